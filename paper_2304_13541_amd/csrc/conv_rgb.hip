// Direct convolution of a 3-channel (RGB) image: the stems of the CNNs of
// Sec. 3 (ResNet-50 7x7/2 -> 64, MobileNetV2 3x3/2 -> 32, VGG-19 3x3/1 -> 64,
// the tiny CNN's 3x3/1 -> 16), fused with scale, shift and activation, on the
// matrix cores.
//
// The image is read as it is (no packing to 8 channels in HBM).  The GEMM
// depth is (window position q, channel c) with c in 0..3 (channel 3 zero), so
// one MFMA depth step of 32 covers 8 window positions and a lane's 8-value
// fragment is two whole pixels: two 8-byte LDS reads for the image operand and
// for the [K][R][R][4] weight operand.
//
// A block takes a strip of consecutive output rows of one image: its input
// rows go to LDS once, widened to 4 channels, with the zero padding around
// them (so the loop tests nothing), and its weight fragments stay in
// registers.  After the one barrier every wave runs its groups of 16 pixels
// on its own: v_mfma_f32_16x16x32_bf16 (rows = output channels, columns =
// pixels), then the group's 16 x K outputs through the wave's own LDS region
// to leave in 16-byte pieces of consecutive addresses.
//
// Bound by instruction issue at two waves per SIMD (7x7: a group's 28 MFMAs
// and about as many cycles of address, scale and packing instructions; the
// waves issue 0.35 of their cycles, wait to issue 0.34 and on dependencies
// 0.31, the matrix cores are busy 0.25) and by each block's start (weights and
// rows, about 3 us); the 3x3 stems by writing the output.  The strip length gives every CU the same number of
// strips, two blocks per CU (7x7) or four (3x3).  Measured against blocks of
// 256 pixels that staged their rows and weights each: 16 images of 224x224
// through the 7x7/2 stem on 128 CUs 26.8 -> 16.7 us (1.8 TB/s), one image on
// 256 CUs 7.3 -> 5.2 us, 8 images through the 3x3/1 stem of 64 channels 15.4
// -> 12.6 us (4.3 TB/s), 32 through the 3x3/2 stem of 32 channels on 128 CUs
// 16.0 -> 12.2 us.
#include <algorithm>

#include "common.hpp"

namespace dstack {

struct RgbArgs {
  const uint16_t* x;  // [N][H][W][3] bf16
  const bf16* w4;     // [K][R][R][4]
  const float* scale;
  const float* shift;
  bf16* y;            // [N][Ho][Wo][K]
  int H, W, Ho, Wo, stride, pad, act;
  int rows;           // output rows of a strip
  int strips;         // strips per image
  int lp, pw;         // LDS row: left zero pixels (even, >= pad), width in pixels (even)
  int vec16;          // W % 8 == 0 and a 16-byte aligned image
  FastDiv div_strips, div_wo, div_units, div_side;
};

constexpr int RGB_LDS = 64 * 1024;  // most bytes of a block's LDS (two blocks per CU)

template <int R, int K>
__global__ __launch_bounds__(256) void conv_rgb_kernel(RgbArgs a) {
  constexpr int RR = R * R;
  constexpr int DC = (RR + 7) / 8;  // depth steps of 8 window positions
  constexpr int KB = K / 16;        // 16-channel MFMA row blocks
  constexpr int ROW = K * 2 + 16;   // staged output row (one pixel), padded against bank conflicts
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  __shared__ __attribute__((aligned(16))) float bnl[2 * K];  // scale, shift
  __shared__ __attribute__((aligned(16))) unsigned char ostage[4][16 * ROW];
  uint2* const patch = reinterpret_cast<uint2*>(smem);  // [input rows][pw] pixels, 4 bf16 each

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, quad = lane >> 4, col = lane & 15;
  const int n = a.div_strips.div(blockIdx.x);
  const int ho0 = (blockIdx.x - n * a.strips) * a.rows;
  const int orows = min(a.rows, a.Ho - ho0);
  const int nrows = (orows - 1) * a.stride + R;  // input rows of the strip, from hi0
  const int hi0 = ho0 * a.stride - a.pad;
  const uint16_t* img = a.x + (long)n * a.H * a.W * 3;

  // Every global load of the start is issued before the first LDS store: the
  // weights (coalesced; the fragments are read back from LDS) and the first
  // round of input rows, so that a block waits for memory once.
  constexpr bool STAGED = R == 7;  // (a 3x3 window's 18 K bytes of weights: straight from memory)
  constexpr int WPT = STAGED ? (K * RR + 255) / 256 : 1;  // weight pixels per thread
  uint2 wv[WPT];
  if (STAGED) {
#pragma unroll
    for (int i = 0; i < WPT; ++i) {
      const int idx = tid + i * 256;
      wv[i] = idx < K * RR ? reinterpret_cast<const uint2*>(a.w4)[idx] : uint2{0u, 0u};
    }
  }
  const float bnv = tid < 2 * K ? (tid < K ? a.scale[tid] : a.shift[tid - K]) : 0.0f;

  // the strip's input rows, widened; rows outside the image are zero
  constexpr int UPT = R == 7 ? 3 : 2;  // 8-pixel units per thread and round
  const int units = a.vec16 ? a.W >> 3 : a.W, total = nrows * units;
  uint4 v[UPT][3];
  auto load_rows = [&](int u0) __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < UPT; ++k) {
      const int u = min(u0 + k * 256, total - 1);
      const int r = a.div_units.div(u), g = u - r * units;
      const int hi = min(max(hi0 + r, 0), a.H - 1);
      const uint4* src = reinterpret_cast<const uint4*>(img + ((long)hi * a.W + 8 * g) * 3);
#pragma unroll
      for (int e = 0; e < 3; ++e) v[k][e] = src[e];
    }
  };
  auto store_rows = [&](int u0) __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < UPT; ++k) {
      const int u = u0 + k * 256;
      if (u >= total) break;
      const int r = a.div_units.div(u), g = u - r * units;
      const bool in = (unsigned)(hi0 + r) < (unsigned)a.H;
      const uint32_t d[12] = {v[k][0].x, v[k][0].y, v[k][0].z, v[k][0].w, v[k][1].x, v[k][1].y,
                              v[k][1].z, v[k][1].w, v[k][2].x, v[k][2].y, v[k][2].z, v[k][2].w};
      uint32_t w[16];  // pixel j -> (c0 | c1 << 16, c2)
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int e = 3 * j;  // first element of pixel j; dword e / 2
        if ((j & 1) == 0) {
          w[2 * j] = d[e / 2];
          w[2 * j + 1] = d[e / 2 + 1] & 0xffffu;
        } else {
          w[2 * j] = (d[e / 2] >> 16) | (d[e / 2 + 1] << 16);
          w[2 * j + 1] = d[e / 2 + 1] >> 16;
        }
      }
      uint4* o = reinterpret_cast<uint4*>(patch + r * a.pw + a.lp + 8 * g);
#pragma unroll
      for (int q = 0; q < 4; ++q)
        o[q] = in ? uint4{w[4 * q], w[4 * q + 1], w[4 * q + 2], w[4 * q + 3]} : uint4{0u, 0u, 0u, 0u};
    }
  };
  if (a.vec16) load_rows(tid);
  if (STAGED) {
#pragma unroll
    for (int i = 0; i < WPT; ++i)
      if (tid + i * 256 < K * RR) patch[tid + i * 256] = wv[i];
    __syncthreads();
  }
  if (tid < 2 * K) bnl[tid] = bnv;
  const uint2* const wsrc = STAGED ? patch : reinterpret_cast<const uint2*>(a.w4);
  // weight fragments: row k = kb*16 + lane%16, window positions q0, q0+1
  bf16x8 wf[KB][DC];
#pragma unroll
  for (int kb = 0; kb < KB; ++kb)
#pragma unroll
    for (int dc = 0; dc < DC; ++dc) {
      const int q0 = dc * 8 + quad * 2;
      const uint2* src = wsrc + (kb * 16 + col) * RR + q0;
      const uint2 v0 = q0 < RR ? src[0] : uint2{0u, 0u};
      const uint2 v1 = q0 + 1 < RR ? src[1] : uint2{0u, 0u};
      wf[kb][dc] = __builtin_bit_cast(bf16x8, uint4{v0.x, v0.y, v1.x, v1.y});
    }
  if (STAGED) __syncthreads();  // the weights' LDS becomes the patch
  if (a.vec16) {  // 8 pixels = 3 16-byte loads -> 4 16-byte LDS writes
    store_rows(tid);
    for (int u0 = tid + UPT * 256; u0 < total; u0 += UPT * 256) {
      load_rows(u0);
      store_rows(u0);
    }
  } else {
    for (int i0 = tid; i0 < total; i0 += 256 * 4) {
      uint32_t c0[4], c1[4], c2[4];
      int dst[4];
      bool in[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int i = min(i0 + k * 256, total - 1);
        const int r = a.div_units.div(i), w = i - r * a.W;
        const int hi = hi0 + r;
        in[k] = (unsigned)hi < (unsigned)a.H;
        dst[k] = r * a.pw + a.lp + w;
        const uint16_t* src = img + ((long)(in[k] ? hi : 0) * a.W + w) * 3;
        c0[k] = src[0];
        c1[k] = src[1];
        c2[k] = src[2];
      }
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (i0 + k * 256 < total) patch[dst[k]] = in[k] ? uint2{c0[k] | (c1[k] << 16), c2[k]} : uint2{0u, 0u};
    }
  }
  {  // zero pixels left and right of every row
    const int side = a.pw - a.W;
    for (int i = tid; i < nrows * side; i += 256) {
      const int r = a.div_side.div(i), s = i - r * side;
      patch[r * a.pw + (s < a.lp ? s : a.W + s)] = uint2{0u, 0u};
    }
  }
  __syncthreads();

  const float lo_clamp = a.act == ACT_NONE ? -INFINITY : 0.0f, hi_clamp = a.act == ACT_RELU6 ? 6.0f : INFINITY;
  // patch offset of this lane's window positions q = dc*8 + quad*2 + h; the
  // depth tail is not a position (its weights are zero and so must its pixels be)
  int qoff[DC][2];
  bool qlast[2];
#pragma unroll
  for (int dc = 0; dc < DC; ++dc)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int q = dc * 8 + quad * 2 + h;
      const int r = q / R, s = q - (q / R) * R;
      qoff[dc][h] = q < RR ? r * a.pw + s : 0;
      if (dc == DC - 1) qlast[h] = q < RR;
    }
  const int npix = orows * a.Wo;
  uint4* const out = reinterpret_cast<uint4*>(a.y + ((long)n * a.Ho + ho0) * a.Wo * K);
  unsigned char* const ot = ostage[wave];
  const uint2* const base = patch + (a.lp - a.pad);
  constexpr int CPP = K / 8;  // 16-byte chunks per pixel
  // scale and shift of the lane's channels: in registers where the weights
  // leave two waves per SIMD anyway, else read from LDS at each use
  constexpr bool BN_REGS = R == 7;
  f32x4 scr[KB], shr[KB];
  auto bn = [&](int kb, f32x4& sc, f32x4& sh) __attribute__((always_inline)) {
    sc = *reinterpret_cast<const f32x4*>(bnl + kb * 16 + 4 * quad);
    sh = *reinterpret_cast<const f32x4*>(bnl + K + kb * 16 + 4 * quad);
  };
  if (BN_REGS) {
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) bn(kb, scr[kb], shr[kb]);
  }
#pragma unroll 1
  for (int g = wave * 16; g < npix; g += 64) {
    const int p = min(g + col, npix - 1);
    const int r = a.div_wo.div(p), wo = p - r * a.Wo;
    const uint2* pp = base + r * a.stride * a.pw + wo * a.stride;
    bf16x8 b[DC];
#pragma unroll
    for (int dc = 0; dc < DC; ++dc) {
      uint2 v[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        v[h] = pp[qoff[dc][h]];
        if (dc == DC - 1 && DC * 8 > RR && !qlast[h]) v[h] = uint2{0u, 0u};
      }
      b[dc] = __builtin_bit_cast(bf16x8, uint4{v[0].x, v[0].y, v[1].x, v[1].y});
    }
    // depth outer, channel blocks inner: KB independent accumulation chains in flight
    f32x4 acc[KB];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) acc[kb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int dc = 0; dc < DC; ++dc)
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) acc[kb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[kb][dc], b[dc], acc[kb], 0, 0, 0);
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
      f32x4 sc = scr[kb], sh = shr[kb];
      if (!BN_REGS) bn(kb, sc, sh);
      float o[4];  // this lane's channels kb*16 + 4*quad.. of its pixel
#pragma unroll
      for (int i = 0; i < 4; ++i) o[i] = __builtin_amdgcn_fmed3f(acc[kb][i] * sc[i] + sh[i], lo_clamp, hi_clamp);
      *reinterpret_cast<uint2*>(ot + col * ROW + (kb * 16 + 4 * quad) * 2) = uint2{pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3])};
    }
    // the wave reads back what its own lanes wrote (LDS keeps a wave's order)
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const int chunks = min(16, npix - g) * CPP;
#pragma unroll
    for (int c0 = 0; c0 < 16 * CPP; c0 += 64) {
      const int c = c0 + lane;
      if (c < chunks) out[g * CPP + c] = *reinterpret_cast<const uint4*>(ot + (c / CPP) * ROW + (c % CPP) * 16);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
}

template <int R, int K>
static dstack_status rgb_launch(const bf16* x, int N, int H, int W, const bf16* w4, int stride, int pad,
                                const float* scale, const float* shift, int act, bf16* y, int Ho, int Wo, int n_cu,
                                hipStream_t st) {
  // widths this entry point takes: the input rows of 256 consecutive output
  // pixels, plus the weights or an output tile of those pixels, in 64 KB
  const int out_rows = (256 + Wo - 2) / Wo + 1;
  const long rows256 = ((long)((out_rows - 1) * stride + R) * W * 8 + 15) / 16 * 16;
  DS_CHECK(rows256 + std::max((long)K * R * R * 8, 256L * (K * 2 + 16)) <= 64 * 1024, DSTACK_E_UNSUPPORTED,
           "conv2d_rgb: image rows too wide for the LDS tile");
  DS_CHECK(((uintptr_t)w4 & 7) == 0 && ((uintptr_t)y & 15) == 0 && ((uintptr_t)scale & 15) == 0 &&
               ((uintptr_t)shift & 15) == 0,
           DSTACK_E_INVALID, "conv2d_rgb: w4 must be 8-byte aligned; y, scale and shift 16-byte aligned");
  RgbArgs a;
  a.x = reinterpret_cast<const uint16_t*>(x); a.w4 = w4; a.scale = scale; a.shift = shift; a.y = y;
  a.H = H; a.W = W; a.Ho = Ho; a.Wo = Wo; a.stride = stride; a.pad = pad; a.act = act;
  a.vec16 = (W % 8 == 0 && ((uintptr_t)x & 15) == 0) ? 1 : 0;
  a.lp = pad + (pad & 1);
  // the last window ends (Wo - 1) * stride + R - pad pixels from the row's start
  const int right = std::max(0, (Wo - 1) * stride + R - pad - W);
  a.pw = (a.lp + W + right + 1) / 2 * 2;
  // strips: as many as fill the CUs k times, for the least k whose strips fit the LDS
  const int fixed = 2 * K * 4 + 4 * 16 * (K * 2 + 16);
  const int max_rows = std::max(1, ((RGB_LDS - fixed) / (a.pw * 8) - R) / stride + 1);
  const long slots = (R == 7 ? 2 : 4) * (long)n_cu;
  for (int k = 1;; ++k) {
    a.rows = ceil_div(Ho, (int)std::max<long>(1, std::min<long>(Ho, k * slots / N)));
    if (a.rows <= max_rows) break;
  }
  a.strips = ceil_div(Ho, a.rows);
  a.div_strips = FastDiv::make(a.strips);
  a.div_wo = FastDiv::make(Wo);
  a.div_units = FastDiv::make(a.vec16 ? W / 8 : W);
  a.div_side = FastDiv::make(std::max(1, a.pw - W));
  // the weights pass through the patch's LDS first
  const size_t lds = std::max((size_t)((a.rows - 1) * stride + R) * a.pw * 8, R == 7 ? (size_t)K * R * R * 8 : 0);
  launch(conv_rgb_kernel<R, K>, dim3((unsigned)(N * a.strips)), dim3(256), lds, st, a);
  return DSTACK_OK;
}

dstack_status launch_conv2d_rgb(const bf16* x, int N, int H, int W, const bf16* w4, int K, int R, int stride, int pad,
                                const float* scale, const float* shift, int act, bf16* y, int n_cu, hipStream_t st) {
  DS_CHECK(N > 0 && H > 0 && W > 0 && stride > 0 && pad >= 0 && pad < R, DSTACK_E_INVALID, "conv2d_rgb: bad shape");
  DS_CHECK(scale && shift, DSTACK_E_INVALID, "conv2d_rgb: scale and shift are required");
  const bool ok = (R == 3 && (K == 16 || K == 32 || K == 64)) || (R == 7 && K == 64);
  DS_CHECK(ok, DSTACK_E_UNSUPPORTED, "conv2d_rgb: supported (R, K): (3, 16), (3, 32), (3, 64), (7, 64)");
  const int Ho = out_dim(H, R, stride, pad), Wo = out_dim(W, R, stride, pad);
  DS_CHECK(Ho > 0 && Wo > 0, DSTACK_E_INVALID, "conv2d_rgb: empty output");
  DS_CHECK((long)N * H * W * 3 < (1L << 31) && (long)N * Ho * Wo * K < (1L << 31), DSTACK_E_UNSUPPORTED,
           "conv2d_rgb: tensor too large");
  dstack_status s;
  if (R == 7)
    s = rgb_launch<7, 64>(x, N, H, W, w4, stride, pad, scale, shift, act, y, Ho, Wo, n_cu > 0 ? n_cu : 256, st);
  else if (K == 16)
    s = rgb_launch<3, 16>(x, N, H, W, w4, stride, pad, scale, shift, act, y, Ho, Wo, n_cu > 0 ? n_cu : 256, st);
  else if (K == 32)
    s = rgb_launch<3, 32>(x, N, H, W, w4, stride, pad, scale, shift, act, y, Ho, Wo, n_cu > 0 ? n_cu : 256, st);
  else
    s = rgb_launch<3, 64>(x, N, H, W, w4, stride, pad, scale, shift, act, y, Ho, Wo, n_cu > 0 ? n_cu : 256, st);
  if (s != DSTACK_OK) return s;
  DS_HIP(hipGetLastError());
  return DSTACK_OK;
}

}  // namespace dstack
