// bf16 implicit-GEMM convolution / linear layer for gfx950 (CDNA4).
//
// A sub-network of the compiled dynamic network is conditional-free tensor
// code (Sec. 5.3); its convolutions and linear layers are dense
// contractions:
//   y[m, co] = sum_{kh, kw, ci} x[img, oh*s - p + kh, ow*s - p + kw, ci] * w[co, kh, kw, ci]
// with m = (img, oh, ow) running over the rows active in this branch.
// As a GEMM: M = rows * Ho * Wo, N = Cout, K = kh * kw * Cin.  NHWC keeps
// the Cin run of one tap contiguous, so A is gathered in 16-byte vectors
// straight from the activation tensor (no im2col buffer).
//
// Workgroup: 64*WM*WN threads computing a BM x BN tile; wave (wm, wn)
// accumulates a (BM/WM) x (BN/WN) block with v_mfma_f32_32x32x16_bf16
// (fp32 accumulate).  K advances 64 per step: the next step's A/B vectors
// are loaded into registers while the current step's MFMAs run from LDS
// (rows padded by 16 bytes: the lanes of each ds_read_b128 phase hit
// distinct banks).  LDS use (<= 55 KB) and registers leave room for two
// workgroups per CU, whose barrier phases interleave.
//
// Tiles are visited in an XCD-aware order: the dispatcher deals workgroups
// round-robin over the 8 XCDs, so consecutive tile indices (the N tiles of
// one M tile, which share their A rows) are given to workgroups of the same
// XCD and its L2.
//
// Epilogue: folded BatchNorm scale/shift (or bias), residual, ReLU or exact
// GELU, then round-to-nearest-even bf16 or an fp32 store.
#include <stdexcept>
#include <type_traits>

#include "conv_dev.hpp"
#include "kernels.hpp"

namespace dycl {
namespace k {

struct ConvP {
  const uint16_t* src;
  const uint16_t* src2;
  int cin1, cin2;
  int H, W, cin, Ho, Wo, cout, stride, pad;
  int M, K, Kp, cin_log2;
  int mt, nt;
  const int32_t* nc;       // device count of live images (<= nmax) or null
  int nmax;                // images the grid is sized for
  // fused gathers / scatters: image i of the layer reads input image
  // srows[i] and residual image rrows[i] and writes output image drows[i]
  // (null: i)
  const int32_t* srows;
  const int32_t* s2rows;   // image list of src2 (the concatenated input)
  int H2, W2, s2;          // src2: spatial shape and the stride it is read at
  uint32_t src_bytes;      // conv_lds_kernel with scalar taps: size of src
  const int32_t* rrows;
  const int32_t* drows;
  // a folded projection (conv_lds_kernel, no K split): its kfold K steps
  // (the last ones of the packed layout) run first; then every sum becomes
  // bf16(fsp * acc + fbp) * finv, the rounded projection output in the
  // units of the block's own sum, which the remaining steps add to
  const float* cell_in;    // ACT_LSTM: old cell state [rows][cout / 4] (through rrows), or null
  float* cell_out;         // ACT_LSTM: new cell state [rows][cout / 4] (through drows)
  int kfold;
  const float* fsp;
  const float* fbp;
  const float* finv;
  int ksplit;              // K ranges per tile (conv_lds_kernel); > 1: fp32 partials to `part`
  float* part;             // [ksplit][M][cout] partial sums (rows of the nmax images)
  const uint16_t* w;
  const float* scale;
  const float* shift;
  const uint16_t* res;
  void* dst;
  int act, out_f32;
  const uint16_t* zeros;   // >= 16 zero bytes: the source of padding taps
  float* gap;              // conv_lds_kernel: 32-row chunk column sums of the bf16 output, or null
  int rev;                 // conv_lds_kernel: each XCD walks its tiles last to first
};

template <int BM, int BN, int WM, int WN, int KS, bool SCALAR, int BK = 64, int STAGES = 1>
__global__ __launch_bounds__(64 * WM* WN) void conv_kernel(ConvP p) {
  constexpr int NT = 64 * WM * WN;
  constexpr int LDK = BK + 8;
  constexpr int VPR = BK / 8;        // 16-byte vectors per tile row
  constexpr int RPP = NT / VPR;      // tile rows per load pass
  constexpr int PA = (BM + RPP - 1) / RPP;
  constexpr int PB = (BN + RPP - 1) / RPP;
  constexpr int WTM = BM / WM, WTN = BN / WN;
  constexpr int TM = WTM / 32, TN = WTN / 32;
  static_assert(TM >= 1 && TN >= 1 && WTM % 32 == 0 && WTN % 32 == 0, "wave tile must be 32x32 blocks");

  __shared__ __align__(16) uint16_t As[STAGES][BM * LDK];
  __shared__ __align__(16) uint16_t Bs[STAGES][BN * LDK];

  // XCD-aware tile order (bijective on [0, mt*nt))
  // with a device count, only the tiles of the live images exist: the
  // grid was sized for nmax images and the surplus workgroups leave
  const int M = p.nc ? min(*p.nc, p.nmax) * p.Ho * p.Wo : p.M;
  const int T = (p.nc ? (M + BM - 1) / BM : p.mt) * p.nt;
  const int T8 = (T >> 3) << 3;
  const int wg = blockIdx.x;
  if (wg >= T) return;
  const int t = wg < T8 ? (wg & 7) * (T8 >> 3) + (wg >> 3) : wg;
  const int mtile = t / p.nt;
  const int m0 = mtile * BM, n0 = (t - mtile * p.nt) * BN;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WN, wn = wave % WN;
  const int chunk = tid % VPR, rsub = tid / VPR;
  const int HoWo = p.Ho * p.Wo;

  // per A row: pixel index of the window origin and its (ih0, iw0); rows
  // past M get an origin far outside the image, so every tap reads zero
  int a_pix[PA], a_pix2[PA], a_ih[PA], a_iw[PA];
#pragma unroll
  for (int i = 0; i < PA; ++i) {
    const int m = m0 + rsub + i * RPP;
    if (m < M) {
      const int img = m / HoWo;
      const int rem = m - img * HoWo;
      const int oh = rem / p.Wo, ow = rem - (rem / p.Wo) * p.Wo;
      const int simg = p.srows ? p.srows[img] : img;
      const int s2img = p.s2rows ? p.s2rows[img] : img;
      a_ih[i] = oh * p.stride - p.pad;
      a_iw[i] = ow * p.stride - p.pad;
      a_pix[i] = (simg * p.H + a_ih[i]) * p.W + a_iw[i];
      a_pix2[i] = (s2img * p.H2 + a_ih[i] * p.s2) * p.W2 + a_iw[i] * p.s2;
    } else {
      a_ih[i] = -0x4000;
      a_iw[i] = -0x4000;
      a_pix[i] = 0;
      a_pix2[i] = 0;
    }
  }

  uint4 ra[PA], rb[PB];
  f32x16 acc[TM][TN];
#pragma unroll
  for (int a = 0; a < TM; ++a)
#pragma unroll
    for (int b = 0; b < TN; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.f;


  auto load_tile = [&](int kt) __attribute__((always_inline)) {
    const int kidx = kt * BK + chunk * 8;
    if constexpr (!SCALAR) {
      int tap = 0, ci = kidx;
      if constexpr (KS != 1) {
        tap = kidx >> p.cin_log2;
        ci = kidx & (p.cin - 1);
      }
      const int kh = tap / KS, kw = tap - (tap / KS) * KS;
      const bool kok = kidx < p.K;
      const uint16_t* sp = p.src;
      int cs = p.cin1, co = ci;
      if (ci >= p.cin1) {
        sp = p.src2;
        cs = p.cin2;
        co = ci - p.cin1;
      }
      const int doff = kh * p.W + kw;
#pragma unroll
      for (int i = 0; i < PA; ++i) {
        uint4 v = make_uint4(0, 0, 0, 0);
        const int ih = a_ih[i] + kh, iw = a_iw[i] + kw;
        if (kok && (unsigned)ih < (unsigned)p.H && (unsigned)iw < (unsigned)p.W && rsub + i * RPP < BM)
          v = *reinterpret_cast<const uint4*>(sp + (size_t)((ci >= p.cin1 ? a_pix2[i] : a_pix[i]) + doff) * cs + co);
        ra[i] = v;
      }
    } else {
#pragma unroll
      for (int i = 0; i < PA; ++i) {
        uint16_t e[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          e[j] = 0;
          const int kk = kidx + j;
          if (kk < p.K && rsub + i * RPP < BM) {
            const int tap = kk / p.cin;
            const int ci = kk - tap * p.cin;
            const int kh = tap / KS, kw = tap - (tap / KS) * KS;
            const int ih = a_ih[i] + kh, iw = a_iw[i] + kw;
            if ((unsigned)ih < (unsigned)p.H && (unsigned)iw < (unsigned)p.W)
              e[j] = p.src[(size_t)(a_pix[i] + kh * p.W + kw) * p.cin + ci];
          }
        }
        ra[i].x = e[0] | (uint32_t(e[1]) << 16);
        ra[i].y = e[2] | (uint32_t(e[3]) << 16);
        ra[i].z = e[4] | (uint32_t(e[5]) << 16);
        ra[i].w = e[6] | (uint32_t(e[7]) << 16);
      }
    }
#pragma unroll
    for (int i = 0; i < PB; ++i) {
      // written on every path: a register array assigned only under a
      // divergent branch is kept in scratch memory by the compiler
      const int row = rsub + i * RPP;
      uint4 v = make_uint4(0, 0, 0, 0);
      if (BN % RPP == 0 || row < BN) v = *reinterpret_cast<const uint4*>(p.w + (size_t)(n0 + row) * p.Kp + kidx);
      rb[i] = v;
    }
  };

  auto store_tile = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < PA; ++i) {
      const int row = rsub + i * RPP;
      if (row < BM) *reinterpret_cast<uint4*>(&As[buf][row * LDK + chunk * 8]) = ra[i];
    }
#pragma unroll
    for (int i = 0; i < PB; ++i) {
      const int row = rsub + i * RPP;
      if (row < BN) *reinterpret_cast<uint4*>(&Bs[buf][row * LDK + chunk * 8]) = rb[i];
    }
  };

  auto compute = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < BK / 16; ++s) {
      bf16x8 af[TM], bfr[TN];
      const int koff = s * 16 + (lane >> 5) * 8;
#pragma unroll
      for (int a = 0; a < TM; ++a)
        af[a] = *reinterpret_cast<const bf16x8*>(&As[buf][(wm * WTM + a * 32 + (lane & 31)) * LDK + koff]);
#pragma unroll
      for (int b = 0; b < TN; ++b)
        bfr[b] = *reinterpret_cast<const bf16x8*>(&Bs[buf][(wn * WTN + b * 32 + (lane & 31)) * LDK + koff]);
#pragma unroll
      for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b)
          acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[a], bfr[b], acc[a][b], 0, 0, 0);
    }
  };

  const int nk = p.Kp / BK;
  load_tile(0);
  if constexpr (STAGES == 1) {
    // one LDS buffer: store, barrier, prefetch the next step, compute, barrier
    for (int kt = 0; kt < nk; ++kt) {
      if (kt > 0) __syncthreads();    // every wave is done reading the previous step
      store_tile(0);
      __syncthreads();
      if (kt + 1 < nk) load_tile(kt + 1);
      compute(0);
    }
  } else {
    // two LDS buffers: one barrier per step
    store_tile(0);
    __syncthreads();
    for (int kt = 0; kt < nk; ++kt) {
      if (kt + 1 < nk) load_tile(kt + 1);
      compute(kt & 1);
      if (kt + 1 < nk) store_tile((kt + 1) & 1);
      __syncthreads();
    }
  }

  // epilogue: lane owns column (lane & 31) of each 32x32 block, rows
  // 8*(r/4) + 4*(lane/32) + r%4
#pragma unroll
  for (int b = 0; b < TN; ++b) {
    const int col = n0 + wn * WTN + b * 32 + (lane & 31);
    if (col >= p.cout) continue;
    const float sc = p.scale ? p.scale[col] : 1.0f;
    const float sh = p.shift ? p.shift[col] : 0.0f;
#pragma unroll
    for (int a = 0; a < TM; ++a) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = m0 + wm * WTM + a * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
        if (row >= M) continue;
        const size_t o = row_at(p.drows, row, HoWo) * p.cout + col;
        float v = fmaf(acc[a][b][r], sc, sh);
        if (p.res) v += bf2f(p.res[row_at(p.rrows, row, HoWo) * p.cout + col]);
        v = apply_act(v, p.act);
        if (p.out_f32)
          static_cast<float*>(p.dst)[o] = v;
        else
          static_cast<uint16_t*>(p.dst)[o] = f2bf(v);
      }
    }
  }
}


// ------------------------------------------------- direct-to-LDS kernel ----
// Same contraction, with gfx950's global_load_lds_dwordx4: each lane's 16
// bytes go straight from global memory to LDS at (wave base + 16 * lane), so
// tiles need no staging registers and no ds_write.  The LDS row of a tile is
// 128 bytes (64 bf16 of K); its eight 16-byte chunks are stored XOR-swizzled
// (physical chunk = logical ^ ((row >> 1) & 7)), which makes the 16 lanes of
// every ds_read_b128 phase of the MFMA operand reads hit 16 distinct bank
// groups.  The swizzle is applied on the global side: each lane picks the
// global chunk that belongs at its fixed LDS slot.  Padding taps and rows
// past M read a zero buffer.  With NS LDS stages the loads of step k + NS - 1
// are issued between the MFMAs of step k, as are the LDS reads of the next
// sub-step's operands (left to itself the compiler reads an operand, waits
// and runs its one or two MFMAs, and puts a wait for every load in flight
// before each LDS read), with one barrier per step.
// NS 1 is the memory-bound case of few K steps, whose speed follows the
// number of workgroups in flight: its registers are capped for five waves
// per SIMD (four with 128 x 128 and 128 x 256 tiles; one spilled register per
// lane cost 20 %).  The others are capped for two waves per SIMD, or for one
// where the LDS of four waves leaves room for one workgroup only.
constexpr int lds_waves_per_simd(int bm, int bn, int waves, int ns) {
  return ns == 1 ? (bn >= 128 ? 4 : 5) : waves == 4 && 2 * ns * (bm + bn) * 128 > 160 * 1024 ? 1 : 2;
}

template <int BM, int BN, int WM, int WN, int KS, int NS, bool LEAN, bool UNI>
__global__ __launch_bounds__(64 * WM* WN)
    __attribute__((amdgpu_waves_per_eu(lds_waves_per_simd(BM, BN, WM * WN, NS)))) void conv_lds_kernel(ConvP p) {
  constexpr int NT = 64 * WM * WN;
  constexpr int WTM = BM / WM, WTN = BN / WN;
  constexpr int TM = WTM / 32, TN = WTN / 32;
  constexpr int A_BYTES = BM * 128, B_BYTES = BN * 128, STAGE = A_BYTES + B_BYTES;
  constexpr int JA = BM * 8 / NT, JB = BN * 8 / NT;
  constexpr int EPW = WTN + 4;                        // epilogue row stride (floats)
  constexpr int EPI = (NT / 64) * 32 * EPW * 4;
  constexpr int SMEM = NS * STAGE > EPI ? NS * STAGE : EPI;
  static_assert(NS >= 1 && NS <= 8, "LDS stages");
  static_assert(BM * 8 % NT == 0 && BN * 8 % NT == 0 && JB >= 1, "tile rows must fill whole load passes");
  static_assert(NT % 128 == 0, "swizzle assumes NT a multiple of 128");
  static_assert(TM >= 1 && TN >= 1 && WTM % 32 == 0 && WTN % 32 == 0, "wave tile must be 32x32 blocks");

  __shared__ __align__(16) char smem[SMEM];

  // with a device count, only the tiles of the live images exist: the
  // grid was sized for nmax images and the surplus workgroups leave.  With
  // a K split, workgroup wg takes K range wg / T of tile wg % T.
  const int M = p.nc ? min(*p.nc, p.nmax) * p.Ho * p.Wo : p.M;
  const int T = (p.nc ? (M + BM - 1) / BM : p.mt) * p.nt;
  const int T8 = (T >> 3) << 3;
  if (static_cast<int>(blockIdx.x) >= T * p.ksplit) return;
  const int split = blockIdx.x / T;
  const int wg = blockIdx.x - split * T;
  const int t = wg < T8 ? (wg & 7) * (T8 >> 3) + (p.rev ? (T8 >> 3) - 1 - (wg >> 3) : (wg >> 3)) : wg;
  const int mtile = t / p.nt;
  const int m0 = mtile * BM, n0 = (t - mtile * p.nt) * BN;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int lchunk = (tid & 7) ^ ((tid >> 4) & 7);   // logical K chunk this thread loads
  const int rbase = tid >> 3;                        // + j * NT / 8
  const int HoWo = p.Ho * p.Wo;

  // per row group of this thread: the window origin (pixel and row / column;
  // rows past M get an origin far outside the image, so every tap reads zero),
  // and the pixel of src2
  int a_pix[JA], a_pix2[JA], a_ih[JA], a_iw[JA];
#pragma unroll
  for (int j = 0; j < JA; ++j) {
    // (a 1x1 layer on scalar addresses has no padding: there the last row
    // stands in for rows past M, whose sums are not stored)
    const int m = UNI && KS == 1 ? min(m0 + rbase + j * (NT / 8), M - 1) : m0 + rbase + j * (NT / 8);
    if (m < M) {
      const int img = m / HoWo;
      const int rem = m - img * HoWo;
      const int oh = rem / p.Wo, ow = rem - (rem / p.Wo) * p.Wo;
      const int simg = p.srows ? p.srows[img] : img;
      a_ih[j] = oh * p.stride - p.pad;
      a_iw[j] = ow * p.stride - p.pad;
      a_pix[j] = (simg * p.H + a_ih[j]) * p.W + a_iw[j];
      a_pix2[j] = 0;
      if (KS == 1 && p.src2) {
        const int s2img = p.s2rows ? p.s2rows[img] : img;
        a_pix2[j] = (s2img * p.H2 + a_ih[j] * p.s2) * p.W2 + a_iw[j] * p.s2;
      }
    } else {
      a_ih[j] = -0x4000;
      a_iw[j] = -0x4000;
      a_pix[j] = 0;
      a_pix2[j] = 0;
    }
  }

  // this workgroup's K steps: [kb, kb + nk) of the layer's Kp / 64
  const int nk_all = p.Kp / 64;
  const int kb = split * nk_all / p.ksplit;
  const int nk = (split + 1) * nk_all / p.ksplit - kb;

  // A K step's loads: the JA row groups of the input, then the JB of the
  // weights.  UNI: 64 divides the channels of each input tensor, so a step is
  // one tap of one tensor for every lane: scalar bases, 32-bit offsets per
  // lane, and the padding of a 3x3 layer from the buffer's range check (tensors
  // below 2^31 bytes).  Else every lane finds its own tap and tensor, and padding comes
  // from a page of zeros.
  constexpr uint32_t kOut = 0xC0000000u;
  struct Step {
    int kt, tap, kh, kw;
    bool second;
  };
  u32x4 abuf{};
  uint32_t aofs[JA], aofs2[JA];
  if constexpr (UNI) {
    if (KS != 1) abuf = raw_buffer(p.src, p.src_bytes);
#pragma unroll
    for (int j = 0; j < JA; ++j) {
      aofs[j] = static_cast<uint32_t>(a_pix[j]) * (p.cin1 * 2) + lchunk * 16;
      aofs2[j] = static_cast<uint32_t>(a_pix2[j]) * (p.cin2 * 2) + lchunk * 16;
    }
  }
  const uint16_t* const wbase = p.w + (size_t)n0 * p.Kp;
  const uint32_t wofs = static_cast<uint32_t>(rbase * p.Kp + lchunk * 8) * 2;
  auto step_of = [&](int kt) __attribute__((always_inline)) {
    Step r;
    kt += kb;
    // a folded projection's steps (the last kfold of the layout) come first
    if (KS == 1 && p.kfold) kt = kt < p.kfold ? kt + (nk_all - p.kfold) : kt - p.kfold;
    r.kt = kt;
    r.tap = KS == 1 ? 0 : (kt * 64) >> p.cin_log2;
    r.kh = r.tap / KS;
    r.kw = r.tap - r.kh * KS;
    r.second = KS == 1 && kt * 64 >= p.cin1;
    return r;
  };
  auto issue = [&](const Step& r, char* sb, int j) __attribute__((always_inline)) {
    if (j >= JA) {
      const int jb = j - JA;
      load_lds16(wbase + ((size_t)jb * (NT / 8) * p.Kp + r.kt * 64), wofs, sb + A_BYTES + (jb * NT + wave * 64) * 16);
    } else if constexpr (UNI) {
      char* const d = sb + (j * NT + wave * 64) * 16;
      if constexpr (KS == 1) {
        load_lds16(r.second ? p.src2 + (r.kt * 64 - p.cin1) : p.src + r.kt * 64, r.second ? aofs2[j] : aofs[j], d);
      } else {
        const int ih = a_ih[j] + r.kh, iw = a_iw[j] + r.kw;
        const bool ok = (unsigned)ih < (unsigned)p.H && (unsigned)iw < (unsigned)p.W;
        const uint32_t tofs = static_cast<uint32_t>((r.kh * p.W + r.kw) * p.cin + (r.kt * 64 - (r.tap << p.cin_log2))) * 2;
        buffer_lds16(abuf, ok ? aofs[j] + tofs : kOut, 0, d);
      }
    } else {
      const int kidx = r.kt * 64 + lchunk * 8;
      int tap = 0, ci = kidx;
      if constexpr (KS != 1) {
        tap = kidx >> p.cin_log2;
        ci = kidx & (p.cin - 1);
      }
      const int kh = tap / KS, kw = tap - (tap / KS) * KS;
      const int ih = a_ih[j] + kh, iw = a_iw[j] + kw;
      const bool ok = kidx < p.K && (unsigned)ih < (unsigned)p.H && (unsigned)iw < (unsigned)p.W;
      // (only a 1x1 layer has a second source)
      const bool second = KS == 1 && ci >= p.cin1;
      const uint16_t* const g = (second ? p.src2 : p.src) +
                                (size_t)((second ? a_pix2[j] : a_pix[j]) + kh * p.W + kw) * (second ? p.cin2 : p.cin1) +
                                (second ? ci - p.cin1 : ci);
      load_lds16(ok ? g : p.zeros, sb + (j * NT + wave * 64) * 16);
    }
  };

  // A = weights (32 output channels), B = pixels: a lane's sums are 4
  // consecutive channels of one pixel per group (channels 8q + 4 hi .. + 3)
  f32x16 acc[TM][TN];
#pragma unroll
  for (int a = 0; a < TM; ++a)
#pragma unroll
    for (int b = 0; b < TN; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.f;

  const int lsw = (lane >> 1) & 7, hi = lane >> 5;
  const int aadr = (wm * WTM + (lane & 31)) * 128 + ((hi ^ lsw) << 4);
  const int badr = A_BYTES + (wn * WTN + (lane & 31)) * 128 + ((hi ^ lsw) << 4);
  bf16x8 af[2][TM], bfr[2][TN];
  auto fetch = [&](const char* st, int s, int f) __attribute__((always_inline)) {
    if (f < TM)
      af[s & 1][f] = *reinterpret_cast<const bf16x8*>(st + ((aadr ^ (s << 5)) + f * 4096));
    else
      bfr[s & 1][f - TM] = *reinterpret_cast<const bf16x8*>(st + ((badr ^ (s << 5)) + (f - TM) * 4096));
  };
  constexpr int NM = TM * TN, NL = JA + JB;
  // the MFMAs of a step from stage `st`; LDS reads run one sub-step ahead, and
  // with `more` the loads of step r into `ld` go out between the MFMAs
  auto compute = [&](const char* st, auto more, const Step& r, char* ld) __attribute__((always_inline)) {
#pragma unroll
    for (int f = 0; f < TM + TN; ++f) fetch(st, 0, f);
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int i = 0; i < NM; ++i) {
        constexpr int PER = NM > 1 ? (2 * (TM + TN) + NM - 1) / NM : TM + TN;
#pragma unroll
        for (int f = i * PER; f < (i + 1) * PER && f < TM + TN; ++f)
          if (s < 3) fetch(st, s + 1, f);
        __builtin_amdgcn_sched_barrier(0);
        acc[i / TN][i % TN] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[s & 1][i % TN], af[s & 1][i / TN],
                                                                      acc[i / TN][i % TN], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (decltype(more)::value) {
          // NL loads over the first three sub-steps' MFMAs
          constexpr int SLOTS = 3 * NM, PL = (NL + SLOTS - 1) / SLOTS;
          const int q = s * NM + i;
#pragma unroll
          for (int j = q * PL; j < (q + 1) * PL && j < NL; ++j) issue(r, ld, j);
        }
      }
  };
  auto issue_all = [&](int kt, char* sb) __attribute__((always_inline)) {
    const Step r = step_of(kt);
#pragma unroll
    for (int j = 0; j < NL; ++j) issue(r, sb, j);
  };

  // a folded projection: once its K steps are summed, each sum becomes the
  // projection's output as the unfused layer stores it (scale, shift, bf16
  // rounding), divided by the block's scale, so the block's own steps add
  // to it and the epilogue's scale / shift finish the residual sum
  auto fold_round = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int b = 0; b < TN; ++b)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        // one group's vectors at a time: all of them would not fit the
        // registers (channels past the last one read zeros)
        __builtin_amdgcn_sched_barrier(0);
        const uint32_t at = static_cast<uint32_t>(n0 + wn * WTN + 4 * hi) * 4 + (b * 32 + 8 * q) * 4, nb = p.cout * 4;
        const u32x4 sp = buffer_load16(p.fsp, nb, at), bp = buffer_load16(p.fbp, nb, at), iv = buffer_load16(p.finv, nb, at);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int a = 0; a < TM; ++a)
            acc[a][b][4 * q + e] = bf2f(f2bf(fmaf(acc[a][b][4 * q + e], __uint_as_float(sp[e]), __uint_as_float(bp[e])))) *
                                   __uint_as_float(iv[e]);
      }
  };

  const bool partial = !LEAN && p.ksplit > 1;   // raw sums; the split reduction finishes them
  // residual vectors of the rows and 8-channel groups this lane finishes in
  // the epilogue (below)
  constexpr int G = WTN / 8;           // 8-channel groups per row
  constexpr int RPV = 64 / G;          // rows per pass
  constexpr int VI = 32 / RPV;         // passes over a 32-row block
  const int g8 = lane % G, col = n0 + wn * WTN + g8 * 8;
  const bool cok = col < p.cout;
  const int row0 = m0 + wm * WTM + lane / G;   // this lane's row in pass 0 of block 0
  // scale and shift of the eight channels that this lane finishes (past the
  // last channel: zeros), requested ahead of the main loop where there are
  // registers for them
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
  auto load_ss = [&]() __attribute__((always_inline)) {
    if (!partial && p.scale) load8(sc, p.scale);
    if (!partial && p.shift) load8(sh, p.shift);
  };
  if (NS > 1) load_ss();
  uint4 rv[2][VI];
  // LEAN: rows of the tile through buffers that end with the layer's last
  // row, at 32-bit offsets; a channel past the last one gets an offset that
  // no buffer reaches
  const uint32_t tbytes = static_cast<uint32_t>(min(BM, M - m0)) * p.cout * 2;
  const uint32_t tofs = cok ? static_cast<uint32_t>((row0 - m0) * p.cout + col) * 2 : kOut;
  const uint32_t pofs = static_cast<uint32_t>(RPV * p.cout) * 2;   // from one pass to the next
  auto load_res = [&](int a) __attribute__((always_inline)) {
#pragma unroll
    for (int v = 0; v < VI; ++v) {
      if constexpr (LEAN) {
        const u32x4 w = buffer_load16(p.res + static_cast<size_t>(m0) * p.cout, tbytes, tofs + (a * VI + v) * pofs);
        rv[a & 1][v] = make_uint4(w[0], w[1], w[2], w[3]);
      } else {
        const int row = row0 + a * 32 + v * RPV;
        rv[a & 1][v] = (row < M && cok) ? *reinterpret_cast<const uint4*>(p.res + row_at(p.rrows, row, HoWo) * p.cout + col)
                                        : make_uint4(0, 0, 0, 0);
      }
    }
  };

  if constexpr (NS == 1) {
    // one stage, the K steps one after another (one step, or a few on a
    // memory-bound layer): a small LDS footprint, more workgroups per CU,
    // whose number (not the bytes in flight per workgroup) sets the speed
    // of these layers
    for (int kt = 0; kt < nk; ++kt) {
      if (kt) lds_barrier();     // every wave is done reading the stage
      issue_all(kt, smem);
      wait_vm_barrier<0>();
      compute(smem, std::false_type{}, Step{}, nullptr);
      if (kt + 1 == p.kfold) fold_round();
    }
  } else {
    // step kt's stage has landed once at most the NS - 2 steps after it are
    // in flight; the stage that step kt + NS - 1 fills was read in step
    // kt - 1, which every wave finished before the barrier of step kt
#pragma unroll
    for (int i = 0; i < NS - 1; ++i)
      if (i < nk) issue_all(i, smem + i * STAGE);
    int cur = 0, ld = (NS - 1) * STAGE;
    int kt = 0;
    for (; kt + NS - 1 < nk; ++kt) {
      const Step r = step_of(kt + NS - 1);
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((NS - 2) * NL) : "memory");
      compute(smem + cur, std::true_type{}, r, smem + ld);
      cur = cur + STAGE == NS * STAGE ? 0 : cur + STAGE;
      ld = ld + STAGE == NS * STAGE ? 0 : ld + STAGE;
      if (kt + 1 == p.kfold) fold_round();
    }
    for (; kt < nk; ++kt) {
      all_barrier();
      compute(smem + cur, std::false_type{}, Step{}, nullptr);
      cur = cur + STAGE == NS * STAGE ? 0 : cur + STAGE;
      if (kt + 1 == p.kfold) fold_round();
    }
  }

  // epilogue through LDS: each wave stages 32 x WTN raw sums in its own
  // region, then every lane finishes 8 consecutive channels of a row (scale
  // and shift, residual, activation, rounding) and writes them with one
  // 16-byte store.  The residual vectors of a block of rows are requested
  // before the stores of the block before it: loads and stores complete in
  // one order.  A wave's LDS operations run in order, so its staging needs no
  // waits of its own.
  const bool res = p.res && !partial;
  if (NS == 1) load_ss();
  if (res) load_res(0);
  seen_barrier();   // the main loop's last tiles are no longer read
  float* ep = reinterpret_cast<float*>(smem) + wave * 32 * EPW;
  // the activation is chosen once, outside the epilogue's loops
  auto epilogue = [&](auto act_c) __attribute__((always_inline)) {
    constexpr int ACT = decltype(act_c)::value;
#pragma unroll
    for (int a = 0; a < TM; ++a) {
#pragma unroll
      for (int b = 0; b < TN; ++b)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          *reinterpret_cast<float4*>(ep + (lane & 31) * EPW + b * 32 + 8 * q + 4 * hi) =
              make_float4(acc[a][b][4 * q], acc[a][b][4 * q + 1], acc[a][b][4 * q + 2], acc[a][b][4 * q + 3]);
      if (a + 1 < TM && res) load_res(a + 1);
      asm volatile("" ::: "memory");
#pragma unroll
      for (int v = 0; v < VI; ++v) {
        const int rl = v * RPV + lane / G;
        const int row = row0 + a * 32 + v * RPV;
        if (LEAN || (row < M && cok)) {
          const float4 lo = *reinterpret_cast<const float4*>(ep + rl * EPW + g8 * 8);
          const float4 hv = *reinterpret_cast<const float4*>(ep + rl * EPW + g8 * 8 + 4);
          if (!LEAN && partial) {
            float* d = p.part + (size_t)split * p.M * p.cout + (size_t)row * p.cout + col;
            *reinterpret_cast<float4*>(d) = lo;
            *reinterpret_cast<float4*>(d + 4) = hv;
            continue;
          }
          float vv[8] = {lo.x, lo.y, lo.z, lo.w, hv.x, hv.y, hv.z, hv.w};
#pragma unroll
          for (int e = 0; e < 8; ++e) vv[e] = fmaf(vv[e], sc[e], sh[e]);
          if constexpr (ACT == ACT_LSTM) {
            // the 8 values are the gates of cells u and u + 1 (input,
            // forget, cell, output each); cell state float32, h bf16
            const int H = p.cout >> 2, u = col >> 2;
            float2 cp = make_float2(0.f, 0.f);
            if (p.cell_in) cp = *reinterpret_cast<const float2*>(p.cell_in + row_at(p.rrows, row, HoWo) * H + u);
            const float c0 = sigmoidf(vv[1]) * cp.x + sigmoidf(vv[0]) * tanhf(vv[2]);
            const float c1 = sigmoidf(vv[5]) * cp.y + sigmoidf(vv[4]) * tanhf(vv[6]);
            const float h0 = sigmoidf(vv[3]) * tanhf(c0), h1 = sigmoidf(vv[7]) * tanhf(c1);
            const size_t oc = row_at(p.drows, row, HoWo) * H + u;
            *reinterpret_cast<float2*>(p.cell_out + oc) = make_float2(c0, c1);
            *reinterpret_cast<uint32_t*>(static_cast<uint16_t*>(p.dst) + oc) = pack_bf16(h0, h1);
            continue;
          }
          if (p.res) {
            const uint32_t rw[4] = {rv[a & 1][v].x, rv[a & 1][v].y, rv[a & 1][v].z, rv[a & 1][v].w};
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              vv[2 * q] += __uint_as_float(rw[q] << 16);
              vv[2 * q + 1] += __uint_as_float(rw[q] & 0xffff0000u);
            }
          }
#pragma unroll
          for (int q = 0; q < 8; ++q) vv[q] = act_t<ACT>(vv[q]);
          if (!LEAN && p.out_f32) {
            float* d = static_cast<float*>(p.dst) + row_at(p.drows, row, HoWo) * p.cout + col;
            *reinterpret_cast<float4*>(d) = make_float4(vv[0], vv[1], vv[2], vv[3]);
            *reinterpret_cast<float4*>(d + 4) = make_float4(vv[4], vv[5], vv[6], vv[7]);
          } else {
            uint4 ov;
            ov.x = pack_bf16(vv[0], vv[1]);
            ov.y = pack_bf16(vv[2], vv[3]);
            ov.z = pack_bf16(vv[4], vv[5]);
            ov.w = pack_bf16(vv[6], vv[7]);
            if constexpr (LEAN)
              buffer_store16(static_cast<uint16_t*>(p.dst) + static_cast<size_t>(m0) * p.cout, tbytes,
                             tofs + (a * VI + v) * pofs, u32x4{ov.x, ov.y, ov.z, ov.w});
            else
              *reinterpret_cast<uint4*>(static_cast<uint16_t*>(p.dst) + row_at(p.drows, row, HoWo) * p.cout + col) = ov;
            if (p.gap) {
              // the stored values back into the staging rows, for the
              // chunk's column sums below
              const uint32_t ow[4] = {ov.x, ov.y, ov.z, ov.w};
              float* e8 = ep + rl * EPW + g8 * 8;
              *reinterpret_cast<float4*>(e8) = make_float4(__uint_as_float(ow[0] << 16), __uint_as_float(ow[0] & 0xffff0000u),
                                                           __uint_as_float(ow[1] << 16), __uint_as_float(ow[1] & 0xffff0000u));
              *reinterpret_cast<float4*>(e8 + 4) = make_float4(__uint_as_float(ow[2] << 16), __uint_as_float(ow[2] & 0xffff0000u),
                                                               __uint_as_float(ow[3] << 16), __uint_as_float(ow[3] & 0xffff0000u));
            }
          }
        }
      }
      if constexpr (ACT != ACT_LSTM) {
        const int row0 = m0 + wm * WTM + a * 32;   // a 32-row chunk of layer rows
        if (p.gap && !partial && row0 < M) {
          asm volatile("" ::: "memory");   // the wave's own rows: in-order LDS
          // rows before `bnd` belong to the chunk's first image, the rest to
          // the next one (an image has at least 32 rows; rows past M land in
          // the second sum of the last image's chunk, which is never read)
          const int bnd = min(32, (row0 / HoWo + 1) * HoWo - row0);
#pragma unroll
          for (int c0 = 0; c0 < WTN; c0 += 64) {
            const int c = c0 + lane, col = n0 + wn * WTN + c;
            if (c < WTN && col < p.cout) {
              float t0 = 0.f, t1 = 0.f;
              if (bnd == 32) {
#pragma unroll 8
                for (int r = 0; r < 32; ++r) t0 += ep[r * EPW + c];
              } else {
                for (int r = 0; r < bnd; ++r) t0 += ep[r * EPW + c];
                for (int r = bnd; r < 32; ++r) t1 += ep[r * EPW + c];
              }
              float* q = p.gap + static_cast<size_t>(row0 / 32) * 2 * p.cout + col;
              q[0] = t0;
              if (bnd < 32) q[p.cout] = t1;   // read only for a chunk that crosses into the next image
            }
          }
        }
      }
      asm volatile("" ::: "memory");   // the reads stay before the next block's staging
    }
  };
  if (p.act == ACT_RELU)
    epilogue(std::integral_constant<int, ACT_RELU>{});
  else if (p.act == ACT_GELU)
    epilogue(std::integral_constant<int, ACT_GELU>{});
  else if (!LEAN && p.act == ACT_TANH)
    epilogue(std::integral_constant<int, LEAN ? ACT_NONE : ACT_TANH>{});
  else if (!LEAN && p.act == ACT_LSTM)
    epilogue(std::integral_constant<int, LEAN ? ACT_NONE : ACT_LSTM>{});
  else
    epilogue(std::integral_constant<int, ACT_NONE>{});
}

// --------------------------------- 3x3 conv, halo tiles, resident weights ----
// For 3x3 / stride 1 / pad 1 layers with 64 input and 64 output channels,
// and for stems with 8 (padded) input channels and 64 output channels.
// A persistent workgroup walks a contiguous range of 128 x 64 output tiles;
// a tile is R whole output rows of one image (or G whole images when an
// image is smaller than the tile).  The tile's input patch - its rows plus
// one halo row above and below, one zero column left and right - is staged
// in LDS once and the nine taps read shifted windows of it, so each input
// pixel crosses L2 -> LDS about (R + 2) / R times instead of nine.
//
// Eight waves in three roles, one barrier per tile:
//  * four compute waves (2 x 2 over the tile, 64 x 32 each) hold their
//    weights in registers for the whole kernel (36 B fragments per lane:
//    9 taps x 4 K sub-steps of one output column), run the 36 MFMA K steps
//    on the current patch and write the finished bf16 tile (scale / shift,
//    residual, activation, rounding) to an LDS staging buffer;
//  * two loader waves copy the next tile's patch and residual rows from
//    global memory straight into LDS and, before the barrier, wait for them;
//  * two store waves copy the previous tile's staging buffer to global
//    memory with 16-byte stores and never wait for them.
// The memory counter of gfx9 counts loads and stores together; with loads
// and stores in different waves, the one wait per tile covers loads issued
// a whole tile earlier and nothing else.
//
// Patch pixels are stored 144 bytes apart (eight 16-byte K chunks and one
// unused slot): the 16 lanes of a ds_read_b128 phase, 16 consecutive
// pixels, fall on 16 distinct bank groups, and a tap's window is a constant
// byte offset from the lane's base address.  With 8 input channels a pixel
// is one 16-byte K chunk (stored densely), a K sub-step of 16 spans two
// taps - tap 2s in lanes 0-31, 2s + 1 in lanes 32-63 - and nine taps take
// five sub-steps (the tenth tap's weights are zero).
struct Conv3P {
  const uint16_t* src;
  const uint16_t* w;      // [64][Kp] packed, K = tap * cin + ci (Kp = 576, or 128 for 8 channels)
  const float* scale;
  const float* shift;
  const uint16_t* res;
  uint16_t* dst;
  const uint16_t* zeros;
  int n, H, W, cout, act;
  int RS, segs, PW, NP;    // rows per patch segment, segments, patch width, patch pixels
  int tiles, tpi;          // tiles; tiles per image (row mode) or 0 (image mode)
  const int32_t* nc;       // device count of live images (<= n) or null
  // image mode only: image i of the layer is image srows[i] of src, rrows[i]
  // of res, drows[i] of dst (null: i); listed tensors are addressed from
  // their first byte, so their size stays below 2^31 bytes (host check)
  const int32_t* srows;
  const int32_t* rrows;
  const int32_t* drows;
};

constexpr int kW3Patch = 256;                      // patch pixels per buffer
constexpr int kW3RB = 128 * 128;                   // 16384 B: a tile of residual / output rows
// patch bytes per pixel and per buffer, by input channels
constexpr int w3_pxb(int cin) { return cin == 8 ? 16 : 144; }
constexpr int w3_pb(int cin) { return kW3Patch * w3_pxb(cin); }

template <int CIN, int ACT, bool RES>
__global__ __launch_bounds__(512) void conv3_wres_kernel(Conv3P p) {
  constexpr int NL = 128;                          // loader / store threads
  constexpr int PXB = w3_pxb(CIN), kW3PB = w3_pb(CIN);
  constexpr int SLOTS = PXB / 16;                  // 16-byte slots per patch pixel (9 or 1)
  constexpr int JP = kW3Patch * SLOTS / NL;        // patch loads per loader thread (18 or 2)
  constexpr int KP = CIN == 8 ? 128 : 576;         // packed row length
  constexpr int NS = CIN == 8 ? 5 : 36;            // K sub-steps of 16
  __shared__ __align__(16) char smem[2 * kW3PB + 4 * kW3RB + 512];
  char* const pbuf = smem;                         // [2][256 px][144 B]
  char* const rbuf = smem + 2 * kW3PB;             // [2][128 rows][128 B] residual
  char* const sbuf = rbuf + 2 * kW3RB;             // [2][128 rows][128 B] finished bf16 tile

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int HW = p.H * p.W;
  // with a device count the live tiles are dealt over the grid (sized for
  // n images); workgroups left without a tile leave
  const int n = p.nc ? min(*p.nc, p.n) : p.n;
  const int tiles = p.nc ? (p.tpi ? n * p.tpi : (n + p.segs - 1) / p.segs) : p.tiles;
  const int t_begin = static_cast<int>((static_cast<long>(tiles) * blockIdx.x) / gridDim.x);
  const int t_end = static_cast<int>((static_cast<long>(tiles) * (blockIdx.x + 1)) / gridDim.x);
  if (t_begin >= t_end) return;

  auto tile_geom = [&](int t, int& img, int& oh0, int& m0, int& lim) __attribute__((always_inline)) {
    if (p.tpi) {
      img = t / p.tpi;
      oh0 = (t - img * p.tpi) * p.RS;
      m0 = img * HW + oh0 * p.W;
      lim = min(p.RS, p.H - oh0) * p.W;
    } else {
      img = t * p.segs;
      oh0 = 0;
      m0 = img * HW;
      lim = min(p.segs, n - img) * HW;
    }
  };
  // 16-byte chunk position of (row, logical chunk) in a residual / staging
  // row of 128 bytes: XOR with (row >> 1) & 7, so that 16 consecutive rows
  // at one logical chunk fall on 16 distinct bank groups
  auto rsw = [](int row, int c) { return c ^ ((row >> 1) & 7); };

  const int wv = __builtin_amdgcn_readfirstlane(wave);   // the same, known wave-uniform
  if (wv >= 6) {
    // ---------------- store waves: tile t - 1 while tile t is computed ----
    // buffer stores: the tile's rows from m0, at most lim of them (stores
    // to later rows fall outside the buffer and are dropped)
    const int st = tid - 6 * 64;
    for (int t = t_begin; t <= t_end; ++t) {
      lds_barrier();
      if (t == t_begin) continue;
      int img, oh0, m0, lim;
      tile_geom(t - 1, img, oh0, m0, lim);
      const char* sb = sbuf + ((t - 1 - t_begin) & 1) * kW3RB;
      if (p.drows) {
        // listed output: a row's image through drows, offsets from dst's start
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const int u = k * NL + st, row = u >> 3, pos = u & 7;
          const int sg = row / HW, px = row - sg * HW;
          const uint32_t o = row < lim ? static_cast<uint32_t>((p.drows[img + sg] * HW + px) * 128 + rsw(row, pos) * 16)
                                       : 0xC0000000u;
          const u32x4 v = *reinterpret_cast<const u32x4*>(sb + u * 16);
          buffer_store16(p.dst, 0x7fffffffu, o, v);
        }
        continue;
      }
      uint16_t* const dbase = p.dst + (size_t)m0 * 64;
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int u = k * NL + st, row = u >> 3, pos = u & 7;
        const u32x4 v = *reinterpret_cast<const u32x4*>(sb + u * 16);
        buffer_store16(dbase, static_cast<uint32_t>(lim) * 128, row * 128 + rsw(row, pos) * 16, v);
      }
    }
    return;
  }

  if (wv >= 4) {
    // ---------------- loader waves: tile t + 1 while tile t is computed ----
    // Buffer loads straight into LDS.  The patch's buffer spans the tile's
    // image(s); a slot's byte offset is relative to the tile's first output
    // row (row mode: plus oh0 rows, so the halo row above image row 0 wraps
    // to a huge offset and rows past the image exceed the buffer), and
    // slots that never hold data (zero columns, the unused ninth slot, past
    // the patch, image-mode halo rows) get an offset above 2^31: all read as
    // zeros, the convolution's padding.
    const int ld = tid - 4 * 64, lw = wv - 4;
    const int rowb = p.W * CIN * 2, imgb = p.H * rowb;
    uint32_t vofs[JP];
    // listed input (image mode): a slot's segment and its offset inside the
    // image (vseg -1: a slot that never holds data); the row ids of a tile's
    // segments are requested with the previous tile's loads
    int vseg[JP], rid[JP];
#pragma unroll
    for (int j = 0; j < JP; ++j) {
      const int u = j * NL + ld, q = u / SLOTS, ch = u - (u / SLOTS) * SLOTS;
      const int segpix = (p.RS + 2) * p.PW;
      const int sg = q / segpix, rem = q - sg * segpix;
      const int pr = rem / p.PW, pc = rem - (rem / p.PW) * p.PW;
      bool data = q < p.NP && ch < 8 && pc >= 1 && pc <= p.W;
      if (!p.tpi) data = data && pr >= 1 && pr <= p.H;
      vofs[j] = data ? static_cast<uint32_t>(sg * imgb + (pr - 1) * rowb + (pc - 1) * CIN * 2 + ch * 16) : 0xC0000000u;
      vseg[j] = data ? sg : -1;
      if (data) vofs[j] -= static_cast<uint32_t>(sg * imgb);
      if (!p.srows) vofs[j] += data ? static_cast<uint32_t>(sg * imgb) : 0u;
      rid[j] = 0;
    }
    // residual slots (listed residual): segment and pixel of each row
    auto fetch_rids = [&](int t) __attribute__((always_inline)) {
      int img, oh0, m0, lim;
      tile_geom(t, img, oh0, m0, lim);
#pragma unroll
      for (int j = 0; j < JP; ++j) rid[j] = vseg[j] >= 0 && img + vseg[j] < n ? p.srows[img + vseg[j]] : -1;
    };
    if (p.srows) fetch_rids(t_begin);
    for (int t = t_begin; t <= t_end; ++t) {
      if (t < t_end) {
        const int buf = (t - t_begin) & 1;
        int img, oh0, m0, lim;
        tile_geom(t, img, oh0, m0, lim);
        const int nimg = p.tpi ? 1 : min(p.segs, n - img);
        char* pb = pbuf + buf * kW3PB;
        if (p.srows) {
#pragma unroll
          for (int j = 0; j < JP; ++j) {
            const uint32_t o = rid[j] >= 0 ? static_cast<uint32_t>(rid[j]) * imgb + vofs[j] : 0xC0000000u;
            buffer_load_lds16(p.src, 0x7fffffffu, o, (lds_void_ptr)(pb + (j * NL + lw * 64) * 16));
          }
        } else {
          const uint16_t* pbase = p.src + (size_t)img * p.H * p.W * CIN;
          const uint32_t pbytes = static_cast<uint32_t>(nimg) * imgb, tofs = static_cast<uint32_t>(oh0) * rowb;
#pragma unroll
          for (int j = 0; j < JP; ++j)
            buffer_load_lds16(pbase, pbytes, vofs[j] + tofs, (lds_void_ptr)(pb + (j * NL + lw * 64) * 16));
        }
        if (RES) {
          char* rb = rbuf + buf * kW3RB;
          if (p.rrows) {
#pragma unroll
            for (int k = 0; k < 8; ++k) {
              const int u = k * NL + ld, row = u >> 3, pos = u & 7;
              const int sg = row / HW, px = row - sg * HW;
              const uint32_t o = row < lim ? static_cast<uint32_t>((p.rrows[img + sg] * HW + px) * 128 + rsw(row, pos) * 16)
                                           : 0xC0000000u;
              buffer_load_lds16(p.res, 0x7fffffffu, o, (lds_void_ptr)(rb + (k * NL + lw * 64) * 16));
            }
          } else {
            const uint16_t* rbase = p.res + (size_t)m0 * 64;
#pragma unroll
            for (int k = 0; k < 8; ++k) {
              const int u = k * NL + ld, row = u >> 3, pos = u & 7;
              buffer_load_lds16(rbase, static_cast<uint32_t>(lim) * 128, row * 128 + rsw(row, pos) * 16,
                                (lds_void_ptr)(rb + (k * NL + lw * 64) * 16));
            }
          }
        }
        if (p.srows && t + 1 < t_end) fetch_rids(t + 1);
      }
      all_barrier();                      // tile t is in LDS for the compute waves
    }
    return;
  }

  // ---------------- compute waves: tile t ----------------
  // MFMA operands: A = weights (32 output channels of this wave), B = patch
  // pixels, so a lane's results are 4 consecutive channels of one pixel per
  // group: channels wn*32 + 8q + 4*hi .. +3, q = 0..3, of pixel (lane & 31)
  const int wm = wave >> 1, wn = wave & 1, hi = lane >> 5;
  const int co_l = wn * 32 + (lane & 31);
  // B fragments: sub-step k covers K 16k .. 16k + 15 (64 channels: tap k/4,
  // channels 16 (k%4) ..; 8 channels: taps 2k, 2k + 1); this lane's half
  bf16x8 bw[NS];
#pragma unroll
  for (int k = 0; k < NS; ++k)
    bw[k] = *reinterpret_cast<const bf16x8*>(p.w + (size_t)co_l * KP + 16 * k + 8 * hi);
  // scale / shift of the 64 channels, in LDS after the staging buffers
  float* const ssl = reinterpret_cast<float*>(sbuf + 2 * kW3RB);
  if (tid < 64) ssl[tid] = p.scale ? p.scale[tid] : 1.0f;
  else if (tid < 128) ssl[tid] = p.shift ? p.shift[tid - 64] : 0.0f;
  int pix0[2];
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    const int i = wm * 64 + a * 32 + (lane & 31);
    const int sg = i / (p.RS * p.W), r = (i / p.W) - sg * p.RS, c = i - (i / p.W) * p.W;
    pix0[a] = sg < p.segs ? (sg * (p.RS + 2) + r) * p.PW + c : 0;
  }
  // a compiler-visible wait: the fragments are resident before the loop,
  // so no memory wait is placed inside it
  __builtin_amdgcn_s_waitcnt(0);

  lds_barrier();                          // the loaders' first tile
  for (int t = t_begin; t < t_end; ++t) {
    const int buf = (t - t_begin) & 1;
    f32x16 acc[2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[a][r] = 0.f;
    if constexpr (CIN == 8) {
      // sub-step k: this lane's tap 2k + hi (the tenth tap has zero weights)
      const char* pcur = pbuf + buf * kW3PB;
#pragma unroll
      for (int k = 0; k < NS; ++k) {
        const int tap = 2 * k + hi < 9 ? 2 * k + hi : 0;
        const int toff = (tap / 3) * p.PW + (tap % 3);
        bf16x8 af[2];
#pragma unroll
        for (int a = 0; a < 2; ++a) af[a] = *reinterpret_cast<const bf16x8*>(pcur + (pix0[a] + toff) * 16);
#pragma unroll
        for (int a = 0; a < 2; ++a) acc[a] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bw[k], af[a], acc[a], 0, 0, 0);
      }
    } else {
      // lane base addresses of the three tap rows; the tap column and the K
      // chunk are constant offsets
      const char* ab[2][3];
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int dy = 0; dy < 3; ++dy) ab[a][dy] = pbuf + buf * kW3PB + (pix0[a] + dy * p.PW) * 144 + hi * 16;
      bf16x8 af[2][2][2];                   // [slot][step of the pair][a]
      auto fetch = [&](int g, int slot) __attribute__((always_inline)) {
        const int tap = g >> 1, dy = tap / 3, dx = tap % 3;
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
          for (int j = 0; j < 2; ++j)
            af[slot][j][a] = *reinterpret_cast<const bf16x8*>(ab[a][dy] + dx * 144 + (2 * (2 * (g & 1) + j)) * 16);
      };
      fetch(0, 0);
#pragma unroll
      for (int g = 0; g < 18; ++g) {
        if (g + 1 < 18) fetch(g + 1, (g + 1) & 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int a = 0; a < 2; ++a)
            acc[a] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bw[2 * g + j], af[g & 1][j][a], acc[a], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
    }

    // epilogue into this tile's staging buffer (the store waves finished its
    // previous contents, tile t - 2, before the last barrier): 8 bytes =
    // 4 channels per group.  All LDS reads of a step are issued before any
    // is used, so their latencies overlap.
    const char* rb = rbuf + buf * kW3RB;
    char* sb = sbuf + buf * kW3RB;
    float4 sc[4], sh[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      sc[q] = *reinterpret_cast<const float4*>(ssl + wn * 32 + 8 * q + 4 * hi);
      sh[q] = *reinterpret_cast<const float4*>(ssl + 64 + wn * 32 + 8 * q + 4 * hi);
    }
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      const int px = wm * 64 + a * 32 + (lane & 31);
      int off[4];
      uint2 rr[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        off[q] = px * 128 + (rsw(px, wn * 4 + q) << 4) + hi * 8;
        if (RES) rr[q] = *reinterpret_cast<const uint2*>(rb + off[q]);
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        float v[4] = {fmaf(acc[a][4 * q], sc[q].x, sh[q].x), fmaf(acc[a][4 * q + 1], sc[q].y, sh[q].y),
                      fmaf(acc[a][4 * q + 2], sc[q].z, sh[q].z), fmaf(acc[a][4 * q + 3], sc[q].w, sh[q].w)};
        if (RES) {
          v[0] += __uint_as_float(rr[q].x << 16);
          v[1] += __uint_as_float(rr[q].x & 0xffff0000u);
          v[2] += __uint_as_float(rr[q].y << 16);
          v[3] += __uint_as_float(rr[q].y & 0xffff0000u);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = apply_act(v[e], ACT);
        bf16x2 lo = {(__bf16)v[0], (__bf16)v[1]}, hv = {(__bf16)v[2], (__bf16)v[3]};
        *reinterpret_cast<uint2*>(sb + off[q]) =
            make_uint2(__builtin_bit_cast(uint32_t, lo), __builtin_bit_cast(uint32_t, hv));
      }
    }
    lds_barrier();                        // staging written; the next tile has landed
  }
}

// ------------------------------------------------------- K-split sums ----
// y[m, c..c+7] = finish(sum_s part[s][m][c..c+7]) with the splits added in
// order s = 0, 1, ...: scale / shift, residual, activation, bf16 rounding,
// as the single-range epilogue does.
template <int ACT>
__global__ __launch_bounds__(256) void ksplit_finish_kernel(const float* __restrict__ part, int S, int Mb, int cout,
                                                            const int32_t* nc, int nmax, int HoWo,
                                                            const float* __restrict__ scale,
                                                            const float* __restrict__ shift,
                                                            const uint16_t* __restrict__ res,
                                                            uint16_t* __restrict__ dst) {
  const int M = (nc ? min(*nc, nmax) : nmax) * HoWo;
  const int C8 = cout >> 3;
  const size_t i = static_cast<size_t>(blockIdx.x) * 256 + threadIdx.x;
  if (i >= static_cast<size_t>(M) * C8) return;
  const size_t row = i / C8;
  const int c = static_cast<int>(i - row * C8) * 8;
  const size_t o = row * cout + c;
  const size_t stride = static_cast<size_t>(Mb) * cout;
  float4 lo = *reinterpret_cast<const float4*>(part + o), hi = *reinterpret_cast<const float4*>(part + o + 4);
  for (int sp = 1; sp < S; ++sp) {
    const float4 a = *reinterpret_cast<const float4*>(part + sp * stride + o);
    const float4 b = *reinterpret_cast<const float4*>(part + sp * stride + o + 4);
    lo.x += a.x; lo.y += a.y; lo.z += a.z; lo.w += a.w;
    hi.x += b.x; hi.y += b.y; hi.z += b.z; hi.w += b.w;
  }
  float vv[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
#pragma unroll
  for (int q = 0; q < 8; ++q) vv[q] = fmaf(vv[q], scale ? scale[c + q] : 1.0f, shift ? shift[c + q] : 0.0f);
  if (res) {
    const uint4 rv = *reinterpret_cast<const uint4*>(res + o);
    const uint32_t rw[4] = {rv.x, rv.y, rv.z, rv.w};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      vv[2 * q] += __uint_as_float(rw[q] << 16);
      vv[2 * q + 1] += __uint_as_float(rw[q] & 0xffff0000u);
    }
  }
#pragma unroll
  for (int q = 0; q < 8; ++q) vv[q] = act_t<ACT>(vv[q]);
  uint4 ov;
  ov.x = pack_bf16(vv[0], vv[1]);
  ov.y = pack_bf16(vv[2], vv[3]);
  ov.z = pack_bf16(vv[4], vv[5]);
  ov.w = pack_bf16(vv[6], vv[7]);
  *reinterpret_cast<uint4*>(dst + o) = ov;
}

// ------------------------------------------------------------- launch ----

namespace {

struct TileCfg {
  int bm, bn, wm, wn;
};

// register-staged kernel (element-gathering stems, unaligned outputs)
constexpr TileCfg kWide[] = {{128, 128, 2, 2}, {128, 64, 2, 2}, {64, 64, 2, 2}};
constexpr TileCfg kMid[] = {{128, 64, 2, 2}, {64, 64, 2, 2}};
constexpr TileCfg kNarrow[] = {{128, 32, 4, 1}, {64, 32, 2, 1}};

long tiles_of(const TileCfg& c, int M, int cout) {
  return (long)((M + c.bm - 1) / c.bm) * ((cout + c.bn - 1) / c.bn);
}

template <size_t N>
TileCfg choose(const TileCfg (&cs)[N], int M, int cout) {
  for (size_t i = 0; i < N; ++i)
    if (tiles_of(cs[i], M, cout) >= 512) return cs[i];
  return cs[N - 1];
}

template <int BM, int BN, int WM, int WN, int KS, bool SC>
void go(const ConvP& p, hipStream_t s) {
  hipLaunchKernelGGL((conv_kernel<BM, BN, WM, WN, KS, SC, 64, 1>), dim3(p.mt * p.nt), dim3(64 * WM * WN), 0, s, p);
}

template <int KS>
void dispatch_staged(const TileCfg& c, const ConvP& p, hipStream_t s) {
  switch (c.bm * 1000 + c.bn) {
    case 128128: go<128, 128, 2, 2, KS, false>(p, s); break;
    case 128064: go<128, 64, 2, 2, KS, false>(p, s); break;
    case 64064: go<64, 64, 2, 2, KS, false>(p, s); break;
    case 128032: go<128, 32, 4, 1, KS, false>(p, s); break;
    default: go<64, 32, 2, 1, KS, false>(p, s); break;
  }
}

// Tile and stages of the direct-to-LDS kernel.
struct LdsCfg {
  int bm, bn, ns;
};

// The tile rule.  t is the number of 128 x 64 tiles; times in us, measured in
// turn on one card, on both sides of each line.
//
// One stage, the K steps in turn: from 1024 tiles on (four workgroups for every
// CU) their number hides the loads, except where a 1x1 layer's K is deep.  256
// images of 56x56, 64 -> 256 with a residual: 128 x 64 | 128 x 128 | 128 x 256
// 183 | 166 | 167; 182 of 28x28, 128 -> 512 with one 77 | 66 | 74; 35915 rows,
// 128 -> 1024, GELU: 128 x 128 on one stage 37, 128 x 256 on three 52; 4096 rows,
// 1024 -> 2048 (1024 tiles, one round of two stages) 33.8, two 27.1; 2073 rows,
// 1024 -> 4096 (1088) 31.4, two 37.9.  K of 1024 runs on 128 x 256 or 128 x 128
// alike (290 images of 7x7, 1024 -> 1024: 33 | 38; 300 of 14x14, 1024 -> 256 37 |
// 41; 137 of 14x14, 1024 -> 1024 65 | 64; 96 of 46x46, 1024 -> 2048, stride 2 256
// | 234).
//
// Fewer tiles are bound by their chains of K steps and the operand bytes per
// step.  Scalar addresses (uni):
//  * 1x1, cout a multiple of 128, short K: two stages of 64 x 64 below 450 tiles
//    and K <= 256 (3000 rows, 256 -> 1024, GELU: 8.4, 128 x 128 on three 11.2; 264
//    images of 7x7, 1024 -> 256: 15.9, 12.7), one of 128 x 64 from 450 with K <=
//    128 (3017 rows, 64 -> 1536, GELU 9.6, 128 x 128 on two 11.4; 20535 rows, 256
//    -> 384: 11.2, two 10.5).
//  * 1x1, other cout: two stages of 64 x 64 up to 360 tiles in one column (35
//    images of 32x32, 768 -> 64: 13.1, 128 x 64 on three 15.5; 51553 rows, 512 ->
//    64, 403 tiles: 13.4, 12.6), 320 in several (13577 rows, 1024 -> 192, 321
//    tiles: 14.1, 13.2; 11606, 1536 -> 192, 273: 17.7, 18.5), 450 with short K
//    (15874 rows, 64 -> 192: 5.7, 6.2); one stage of 128 x 64 from 512 with K <=
//    512 (5 of 56x56, 256 -> 320: 9.2, three 10.9; 76 of 16x16, 1024 -> 192: 17.1,
//    three 15.2).
//  * 128 x 256, three stages, from 160 of them: 20972 rows x 256, K 1024 (164):
//    18.4, 128 x 128 on three 19.1, 64 x 128 20.9; 3x3, stride 2, K 2304: 32.3,
//    36.4, 37.3.  (The gain over 128 x 128 needs the input in the caches, as a
//    layer's output is for the next one.)
//  * 128 x 128 from 192: three stages up to one workgroup per CU, then two, two
//    per CU (4096 x 1024, K 2048, 256 tiles: 21.7, two stages 28.4, 64 x 128
//    24.6).  64 x 128 from 160: 2499 x 512, K 2048: 14.2, 64 x 64 14.7; 1024 x
//    1024, K 2048, 128 tiles: 14.6, 64 x 64 11.5.
// Addresses per lane take more instructions per step and tiles of their own: 256
// images of 28x28, 480 -> 256: 128 x 128 on one stage 90 (128 x 64 on three 125);
// 64 x 128 on three stages while two workgroups per CU hold them all, else on two,
// three per CU (124 of 22x22, 1000 -> 320, stride 2, 705 tiles: 21.4, three 22.3,
// 64 x 64 28.2; 9 of 32x32, 64 -> 1024, 7x7, stride 2, 288: three 32.0, two 39.7);
// 64 x 64 where half of a 64 x 128 tile can be empty (875 of 7x7, 480 -> 192,
// stride 2: 9.8, 64 x 128 9.8, 128 x 64 on three 10.9).
// Below 64 channels: three stages (60 KB, two workgroups per CU), two where there
// are more tiles than that (1765 images of 56x56, 64 -> 32, stride 2: 64, three
// 96) unless the K is deep (149 of 32x32, 600 -> 32: 40.0, three 34.4; 1018 of
// 42x42, 256 -> 16, 3x3: 1075, 588) or the taps of a 3x3 layer do not overlap
// (1823 of 16x16, 128 -> 16, stride 2: 36.4, 30.5); one for one K step of
// per-lane addresses from 256 tiles, or three from 1024 (2048 images of 32x32,
// stride 2, 16 -> 32: 1x1 18.9, three 31.0, 3x3 15.1, 20.4).
LdsCfg choose_lds(int M, int cout, int Kp, int k, int stride, bool uni) {
  auto tiles = [&](int bm, int bn) { return static_cast<long>((M + bm - 1) / bm) * ((cout + bn - 1) / bn); };
  const long t = tiles(128, 64);
  const bool n128 = cout % 128 == 0;
  if (cout < 64) {
    if (!uni && Kp <= 192 && t >= (Kp == 64 ? 256 : 1024)) return {128, 32, 1};
    const bool shallow = !uni ? Kp <= 512 : k == 1 || (stride == 1 && Kp <= 1152);
    return {128, 32, tiles(128, 32) > 512 && shallow ? 2 : 3};
  }
  if (t >= 1024 && (!uni || k != 1 || Kp <= 256 || (t > 1024 && Kp <= 1024)))
    return uni && k == 1 && cout % 256 == 0 && Kp == 1024 ? LdsCfg{128, 256, 1} : LdsCfg{128, n128 ? 128 : 64, 1};
  if (!uni) {
    const long n = tiles(64, 128);
    const bool whole = n128 || (cout > 64 && Kp > 512 && t >= 256 && (n <= 512 || t >= 512));
    if (whole && n >= 160) return {64, 128, n <= 512 ? 3 : 2};
    if (t >= 512) return {128, 64, 1};
    return {64, 64, t >= 256 ? 2 : 4};
  }
  if (k == 1 && t >= 256) {
    if (n128 ? t < 450 && Kp <= 256 : t < (cout == 64 ? 360 : Kp <= 256 ? 450 : 320)) return {64, 64, 2};
    if (n128 ? t >= 450 && Kp <= 128 : t >= 512 && Kp <= 512) return {128, 64, 1};
  }
  if (cout % 256 == 0 && tiles(128, 256) >= 160) return {128, 256, 3};
  if (n128) {
    const long t128 = tiles(128, 128);
    if (t128 >= 192) return {128, 128, t128 <= 256 ? 3 : 2};
    if (tiles(64, 128) >= 160) return {64, 128, 3};
  } else if (t >= 256) {
    return {128, 64, 3};
  }
  return {64, 64, 4};
}

// LEAN: bf16 output in the layer's own rows, no K split, no cell (fewer
// registers, and stores and residual through range-checked buffers).  UNI:
// scalar taps and sources (below).
template <int BM, int BN, int WM, int WN, int KS, int NS, bool LEAN, bool UNI>
void go_lds(const ConvP& p, hipStream_t s, int S) {
  hipLaunchKernelGGL((conv_lds_kernel<BM, BN, WM, WN, KS, NS, LEAN, UNI>), dim3(p.mt * p.nt * S), dim3(64 * WM * WN), 0,
                     s, p);
}

template <int KS, bool LEAN, bool UNI>
void dispatch_tile(const LdsCfg& c, const ConvP& p, hipStream_t s, int S) {
  switch ((c.bm * 1000 + c.bn) * 10 + c.ns) {
    case 1281281: return go_lds<128, 128, 2, 2, KS, 1, LEAN, UNI>(p, s, S);
    case 1280641: return go_lds<128, 64, 2, 2, KS, 1, LEAN, UNI>(p, s, S);
    case 641283: return go_lds<64, 128, 2, 2, KS, 3, LEAN, UNI>(p, s, S);
    case 640644: return go_lds<64, 64, 2, 2, KS, 4, LEAN, UNI>(p, s, S);
    case 1280322: return go_lds<128, 32, 4, 1, KS, 2, LEAN, UNI>(p, s, S);
    case 1280323: return go_lds<128, 32, 4, 1, KS, 3, LEAN, UNI>(p, s, S);
  }
  if constexpr (!UNI || KS == 1)
    if (c.bm == 64 && c.bn == 64 && c.ns == 2) return go_lds<64, 64, 2, 2, KS, 2, LEAN, UNI>(p, s, S);
  if constexpr (UNI) {
    if (c.bm == 128 && c.bn == 256 && c.ns == 3) return go_lds<128, 256, 2, 4, KS, 3, LEAN, true>(p, s, S);
    if (c.bm == 128 && c.bn == 128 && c.ns == 2) return go_lds<128, 128, 2, 2, KS, 2, LEAN, true>(p, s, S);
    if (c.bm == 128 && c.bn == 128 && c.ns == 3) return go_lds<128, 128, 2, 2, KS, 3, LEAN, true>(p, s, S);
    if (c.bm == 128 && c.bn == 64 && c.ns == 3) return go_lds<128, 64, 2, 2, KS, 3, LEAN, true>(p, s, S);
    if constexpr (KS == 1)
      if (c.bm == 128 && c.bn == 256 && c.ns == 1) return go_lds<128, 256, 2, 4, KS, 1, LEAN, true>(p, s, S);
  } else {
    if (c.bm == 64 && c.bn == 128 && c.ns == 2) return go_lds<64, 128, 2, 2, KS, 2, LEAN, false>(p, s, S);
    if (c.bm == 128 && c.bn == 32 && c.ns == 1) return go_lds<128, 32, 4, 1, KS, 1, LEAN, false>(p, s, S);
  }
  throw std::invalid_argument("conv_bf16: no kernel for this tile");   // (the grid is laid out for the tile)
}

void dispatch_lds(int k, const LdsCfg& c, const ConvP& p, hipStream_t s, int S, bool uni) {
  const bool lean =
      S == 1 && !p.out_f32 && !p.rrows && !p.drows && (p.act == ACT_RELU || p.act == ACT_NONE || p.act == ACT_GELU);
  if (k == 7) dispatch_tile<7, false, false>(c, p, s, S);
  else if (uni && lean) k == 1 ? dispatch_tile<1, true, true>(c, p, s, S) : dispatch_tile<3, true, true>(c, p, s, S);
  else if (uni) k == 1 ? dispatch_tile<1, false, true>(c, p, s, S) : dispatch_tile<3, false, true>(c, p, s, S);
  else if (lean) k == 1 ? dispatch_tile<1, true, false>(c, p, s, S) : dispatch_tile<3, true, false>(c, p, s, S);
  else k == 1 ? dispatch_tile<1, false, false>(c, p, s, S) : dispatch_tile<3, false, false>(c, p, s, S);
}

// Tile geometry of the halo kernels: BM-pixel tiles of R whole rows of one
// image, or of G whole images; the patch (tile rows + halo) must fit `cap`
// pixels.
struct HaloGeom {
  int RS, segs, tpi, PW, NP, mtiles;
};

bool halo_geom(int n, int H, int W, int bm, int cap, HaloGeom& g) {
  if (W > bm || n <= 0) return false;
  const int HW = H * W;
  if (HW > bm) {
    g.RS = bm / W;
    g.segs = 1;
    g.tpi = (H + g.RS - 1) / g.RS;
    g.mtiles = n * g.tpi;
  } else {
    g.RS = H;
    g.segs = bm / HW;
    while (g.segs > 1 && g.segs * (H + 2) * (W + 2) > cap) --g.segs;
    g.tpi = 0;
    g.mtiles = (n + g.segs - 1) / g.segs;
  }
  g.PW = W + 2;
  g.NP = g.segs * (g.RS + 2) * g.PW;
  return g.NP <= cap;
}

int cu_count() {
  static int cus[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 0;
  if (!cus[dev] && hipDeviceGetAttribute(&cus[dev], hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    cus[dev] = 0;
  return cus[dev];
}

bool is_halo_layer(const ConvArgs& a) {
  return a.k == 3 && a.stride == 1 && a.pad == 1 && !a.src2 && !a.out_f32 && a.Ho == a.H && a.Wo == a.W &&
         a.cin % 64 == 0 && a.cout % 64 == 0 && a.Kp == 9 * a.cin &&
         !((reinterpret_cast<uintptr_t>(a.scale) | reinterpret_cast<uintptr_t>(a.shift)) & 15);
}

// the weights-resident 3x3 kernel (64 -> 64 channels)
bool conv3_wres(const ConvArgs& a, hipStream_t s) {
  HaloGeom g;
  const bool stem = a.cin == 8 && a.Kp == 128 && a.k == 3 && a.stride == 1 && a.pad == 1 && !a.src2 && !a.out_f32 &&
                    a.Ho == a.H && a.Wo == a.W &&
                    !((reinterpret_cast<uintptr_t>(a.scale) | reinterpret_cast<uintptr_t>(a.shift)) & 15);
  if (!(stem || (is_halo_layer(a) && a.cin == 64)) || a.cout != 64 || !halo_geom(a.n, a.H, a.W, 128, kW3Patch, g))
    return false;
  const int cus = cu_count();
  if (!cus) return false;
  Conv3P p;
  p.src = a.src;
  p.w = a.w;
  p.scale = a.scale;
  p.shift = a.shift;
  p.res = a.res;
  p.dst = static_cast<uint16_t*>(a.dst);
  p.zeros = a.zeros;
  p.n = a.n;
  p.H = a.H;
  p.W = a.W;
  p.cout = a.cout;
  p.act = a.act;
  p.RS = g.RS;
  p.segs = g.segs;
  p.tpi = g.tpi;
  p.PW = g.PW;
  p.NP = g.NP;
  p.tiles = g.mtiles;
  p.nc = a.ncount;
  // row lists: image mode only, no concatenated input, and every listed
  // tensor small enough for 31-bit byte offsets from its start
  const bool listed = a.src_rows || a.res_rows || a.dst_rows;
  if (listed && (stem || g.tpi != 0 || a.src2_rows || a.list_rows <= 0 ||
                 static_cast<long>(a.list_rows) * a.H * a.W * 128 > 0x7ffffff0L))
    return false;
  p.srows = a.src_rows;
  p.rrows = a.res_rows;
  p.drows = a.dst_rows;
  const int grid = p.tiles < cus ? p.tiles : cus;
  auto go = [&](auto kern) { hipLaunchKernelGGL(kern, dim3(grid), dim3(512), 0, s, p); };
#define DYCL_W(CIN)                                                     \
  if (p.res) {                                                          \
    if (p.act == ACT_RELU) go(conv3_wres_kernel<CIN, ACT_RELU, true>);  \
    else if (p.act == ACT_GELU) go(conv3_wres_kernel<CIN, ACT_GELU, true>); \
    else go(conv3_wres_kernel<CIN, ACT_NONE, true>);                    \
  } else {                                                              \
    if (p.act == ACT_RELU) go(conv3_wres_kernel<CIN, ACT_RELU, false>); \
    else if (p.act == ACT_GELU) go(conv3_wres_kernel<CIN, ACT_GELU, false>); \
    else go(conv3_wres_kernel<CIN, ACT_NONE, false>);                   \
  }
  if (stem) {
    DYCL_W(8)
  } else {
    DYCL_W(64)
  }
#undef DYCL_W
  return true;
}

}  // namespace

__device__ __align__(16) uint16_t g_zero_page[64];   // zero-initialised device memory

const uint16_t* zero_page() {
  static const uint16_t* addr[64] = {nullptr};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
  if (!addr[dev]) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(g_zero_page)) != hipSuccess) return nullptr;
    addr[dev] = static_cast<const uint16_t*>(ptr);
  }
  return addr[dev];
}

int conv_ksplit(int Ho, int Wo, int cout, int K, bool out_f32) {
  // measured: K = 4608 on 4x4 and 7x7 outputs gains from four ranges
  // (ResNet-50 stage 4, 51 images: 42 -> 34 us; ResNet-18 stage 4, 255
  // images: its step 1.218 -> 1.201 ms, same box, interleaved runs), K =
  // 2304 loses from two (the partial sums cost more than the idle CUs)
  if (out_f32 || Ho * Wo > 64 || K < 4608 || cout < 256 || cout % 64) return 1;
  return 4;
}

int conv_cout_pad(int cout) {
  if (cout >= 256) return (cout + 255) / 256 * 256;
  if (cout >= 128) return (cout + 127) / 128 * 128;
  if (cout >= 64) return (cout + 63) / 64 * 64;
  return (cout + 31) / 32 * 32;
}

bool conv_bf16(const ConvArgs& a, hipStream_t s) {
  if (a.pool) return false;   // only conv_rgb_stem fuses a max-pool (its dst is the pooled tensor)
  if (a.cin == 3 && conv_rgb_stem(a, s)) return false;
  ConvP p;
  p.src = a.src;
  p.src2 = a.src2;
  p.H2 = a.src2_H > 0 ? a.src2_H : a.H;
  p.W2 = a.src2_W > 0 ? a.src2_W : a.W;
  p.s2 = a.src2_stride > 0 ? a.src2_stride : 1;
  p.cin1 = a.cin1;
  p.cin2 = a.cin2;
  p.H = a.H;
  p.W = a.W;
  p.cin = a.cin;
  p.Ho = a.Ho;
  p.Wo = a.Wo;
  p.cout = a.cout;
  p.stride = a.stride;
  p.pad = a.pad;
  p.M = a.n * a.Ho * a.Wo;
  p.K = a.k * a.k * a.cin;
  p.Kp = a.Kp;
  int lg = 0;
  while ((1 << lg) < a.cin) ++lg;
  p.cin_log2 = lg;
  p.w = a.w;
  p.scale = a.scale;
  p.shift = a.shift;
  p.res = a.res;
  p.dst = a.dst;
  p.act = a.act;
  p.out_f32 = a.out_f32;
  p.zeros = a.zeros;
  p.nc = a.ncount;
  p.nmax = a.n;
  p.ksplit = 1;
  p.part = nullptr;
  p.cell_in = a.cell_in;
  p.cell_out = a.cell_out;
  p.gap = nullptr;
  p.rev = a.rev;
  p.kfold = a.kfold;
  p.fsp = a.fold_sp;
  p.fbp = a.fold_bp;
  p.finv = a.fold_inv;
  if (a.kfold && (!a.src2 || a.cin1 % kBK || a.cin2 != a.kfold * kBK || a.k != 1 || a.res || a.out_f32 ||
                  !a.fold_sp || !a.fold_bp || !a.fold_inv || a.cout % 8 || (reinterpret_cast<uintptr_t>(a.dst) & 15) ||
                  !a.zeros))
    throw std::invalid_argument("folded projection: arguments the implicit-GEMM kernel does not take");
  // tanh and the LSTM cell exist only in the implicit GEMM's epilogue: a
  // linear layer on 1x1 rows with 16-byte output vectors, never split
  const bool special = a.act == ACT_TANH || a.act == ACT_LSTM;
  if (special && (a.k != 1 || a.H != 1 || a.W != 1 || a.cin % 8 || a.cout % 8 || a.res || a.out_f32 || !a.zeros ||
                  (reinterpret_cast<uintptr_t>(a.dst) & 15) ||
                  (a.act == ACT_LSTM && (!a.cell_out || (reinterpret_cast<uintptr_t>(a.cell_out) & 7) ||
                                         (reinterpret_cast<uintptr_t>(a.cell_in) & 7)))))
    throw std::invalid_argument("tanh / LSTM-cell epilogue: arguments the implicit-GEMM kernel does not take");
  p.srows = a.src_rows;
  p.s2rows = a.src2_rows;
  p.rrows = a.res_rows;
  p.drows = a.dst_rows;

  // 16-byte A vectors need Cin % 8 == 0, and a power-of-two Cin when the tap
  // index is split off with a shift; anything else gathers element by element
  const bool pow2 = (a.cin & (a.cin - 1)) == 0;
  const bool scalar = (a.cin % 8) != 0 || (a.k != 1 && !pow2);
  if (scalar) {
    const TileCfg c = a.cout >= 64 ? TileCfg{128, 64, 2, 2} : TileCfg{128, 32, 4, 1};
    p.mt = (p.M + c.bm - 1) / c.bm;
    p.nt = (a.cout + c.bn - 1) / c.bn;
    if (c.bn == 64) {
      if (a.k == 7) go<128, 64, 2, 2, 7, true>(p, s);
      else if (a.k == 3) go<128, 64, 2, 2, 3, true>(p, s);
      else go<128, 64, 2, 2, 1, true>(p, s);
    } else {
      if (a.k == 7) go<128, 32, 4, 1, 7, true>(p, s);
      else if (a.k == 3) go<128, 32, 4, 1, 3, true>(p, s);
      else go<128, 32, 4, 1, 1, true>(p, s);
    }
    return false;
  }
  // tile shapes follow the expected live rows (the grid covers all n)
  const int Mh = (a.nhint > 0 && a.nhint < a.n ? a.nhint : a.n) * a.Ho * a.Wo;
  // the direct-to-LDS kernel stores 8 channels per 16-byte vector
  const bool vec_out = a.cout % 8 == 0 && (reinterpret_cast<uintptr_t>(a.dst) & 15) == 0 &&
                       (reinterpret_cast<uintptr_t>(a.res) & 15) == 0 && a.zeros != nullptr;
  // the kernel on linear pixel tiles reads contiguous images: a layer with row
  // lists takes the register-weight halo kernel (image mode) or the implicit GEMM
  const bool listed = a.src_rows || a.src2_rows || a.res_rows || a.dst_rows;
  if (conv3_narrow(a, s)) return false;   // 16 / 32 channels: row lists allowed
  // 64 -> 64 channels on few pixels: the tile kernel, whose workgroups start
  // without loading all weights first, while two per CU hold its 128 x 64 tiles
  // (us, register-weight kernel | tiles: 500 images of 8x8 9.4 | 7.9, 300 of 14x14
  // 11.8 | 9.0, 20 of 56x56 (490 tiles) 12.8 | 9.8, 22 of them (539) 12.5 | 13.7; 1078
  // 18.9 | 23.0)
  if (vec_out && !listed && a.cin == 64 && a.cout == 64 && Mh <= 512 * 128 && conv3_tiles(a, s)) return false;
  if (vec_out && (listed ? conv3_wres(a, s) : (conv3_wres(a, s) || conv3_tiles(a, s)))) return false;
  if (vec_out) {
    // deep K on few pixels per image: K ranges of one tile on several
    // workgroups, fp32 partials summed in a fixed order by a second kernel
    // (the split depends on the layer's shape only, never on n)
    const int S = conv_ksplit(a.Ho, a.Wo, a.cout, p.K, a.out_f32 != 0);
    const bool split = S > 1 && a.splitws && !a.res_rows && !a.dst_rows && !a.kfold && !special &&
                       a.splitws_bytes >= static_cast<size_t>(S) * p.M * a.cout * sizeof(float);
    // scalar taps and offsets (UNI): 64 divides the channels of each input
    // tensor, the tensors lie below 2^31 bytes, and a 1x1 layer has no padding
    // (a specification may ask for it; that path reads every pixel unchecked)
    const long b1 = static_cast<long>(a.src_rows ? a.list_rows : a.n) * a.H * a.W * a.cin1 * 2;
    const long b2 = a.src2 ? static_cast<long>(a.src2_rows ? a.src2_list_rows : a.n) * p.H2 * p.W2 * a.cin2 * 2 : 0;
    const bool uni = (a.k == 3 || (a.k == 1 && a.pad == 0)) && a.cin1 % 64 == 0 && (!a.src2 || a.cin2 % 64 == 0) &&
                     b1 < 0x7fffffffL && b2 < 0x7fffffffL && (!a.src_rows || a.list_rows > 0) &&
                     (!a.src2_rows || a.src2_list_rows > 0);
    p.src_bytes = static_cast<uint32_t>(b1);
    // a split layer: 64 x 128 tiles while the four ranges of 128 x 128 tiles
    // leave CUs idle (60 images of 4x4x512: 17 us against 24; 255 images, 512
    // workgroups of 128 x 128: 39 against 42); addresses per lane: up to 512 (7x7,
    // 128 -> 512 on 7x7: 60 images, 368 workgroups, 43, 128 x 128 on one stage 47;
    // 120 images, 736, 74, 67)
    const long t128 = (static_cast<long>(Mh) + 127) / 128 * ((a.cout + 127) / 128);
    const bool few = S * t128 < 256;
    const LdsCfg c = !split         ? choose_lds(Mh, a.cout, p.Kp, a.k, a.stride, uni)
                     : a.cout % 128 ? (uni ? LdsCfg{128, 64, 3} : few ? LdsCfg{64, 64, 2} : LdsCfg{128, 64, 1})
                     : few          ? LdsCfg{64, 128, 3}
                     : uni          ? LdsCfg{128, 128, 2}
                     : S * t128 < 512 ? LdsCfg{64, 128, 3}
                                      : LdsCfg{128, 128, 1};
    p.mt = (p.M + c.bm - 1) / c.bm;
    p.nt = (a.cout + c.bn - 1) / c.bn;
    if (split) {
      p.ksplit = S;
      p.part = a.splitws;
      dispatch_lds(a.k, c, p, s, S, uni);
      const size_t items = static_cast<size_t>(p.M) * (a.cout / 8);
      const dim3 fgrid(static_cast<unsigned>((items + 255) / 256));
      auto finish = [&](auto k) {
        hipLaunchKernelGGL(k, fgrid, dim3(256), 0, s, a.splitws, S, p.M, a.cout, a.ncount, a.n, a.Ho * a.Wo, a.scale,
                           a.shift, a.res, static_cast<uint16_t*>(a.dst));
      };
      if (a.act == ACT_RELU)
        finish(ksplit_finish_kernel<ACT_RELU>);
      else if (a.act == ACT_GELU)
        finish(ksplit_finish_kernel<ACT_GELU>);
      else
        finish(ksplit_finish_kernel<ACT_NONE>);
      return false;
    }
    // (a layer that runs on the linear pixel tiles at other row counts leaves the
    // pooling to the exit as there: a row's sums keep one order)
    if (a.gap_part && !a.out_f32 && !a.dst_rows && a.act != ACT_LSTM && a.Ho * a.Wo >= 32 && !conv3_tiles_shape(a))
      p.gap = a.gap_part;
    dispatch_lds(a.k, c, p, s, 1, uni);
    return p.gap != nullptr;
  }
  const TileCfg c = a.cout >= 128 ? choose(kWide, Mh, a.cout)
                    : a.cout >= 64 ? choose(kMid, Mh, a.cout)
                                   : choose(kNarrow, Mh, a.cout);
  p.mt = (p.M + c.bm - 1) / c.bm;
  p.nt = (a.cout + c.bn - 1) / c.bn;
  if (a.k == 1)
    dispatch_staged<1>(c, p, s);
  else if (a.k == 3)
    dispatch_staged<3>(c, p, s);
  else
    dispatch_staged<7>(c, p, s);
  return false;
}

}  // namespace k
}  // namespace dycl
