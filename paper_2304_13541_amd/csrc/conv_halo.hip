// 3x3 convolutions of stride 1 and padding 1 on gfx950 matrix cores (bf16 in,
// fp32 accumulate): the layers that hold most of the FLOPs of the served CNNs
// (Sec. 3, Sec. 4.1).  Same arithmetic and epilogue as the general implicit
// GEMM: y = act(scale * conv(x, w) + shift [+ res]), NHWC / KRSC.
//
// What bounds the general kernel on these layers is the LDS port (it moves 98
// of the port's 128 bytes per clock and CU on VGG-19's large layers, at 0.25 of
// the MFMA rate): it copies every pixel row into LDS nine times, once per
// window position, and reads it back for the products.  Here a block copies
// the input pixels under its output tile once per 64 channels (the patch:
// the tile and a one-pixel halo, 128-byte rows) and reads the nine windows
// from it; only the weights stream through a ring, 64 deep at a time, one
// window position (tap) per step.  So a 64 x 128 tile moves about 10 KB per
// step into LDS instead of 24 KB, and a 128 x 256 tile 21 KB instead of 48.
//
// Tiles.  BN output channels x BM pixels; either BM consecutive pixels of the
// flattened tensor (then the patch is BM + 2W + 2 consecutive pixels, and
// lanes whose tap leaves the image read a row of zeros), or th x tw pixels of
// one image (patch (th+2) x (tw+2), zeros around the image).  The 64 x 128
// tile runs in blocks of 4 waves with 80 KB of LDS, two to a CU, so that one
// block's start and epilogue (3-4 us of fixed latency) overlap the other's
// products; the 128 x 256 tile runs one block of 8 waves per CU; the 64 x 64
// tile splits each 64-deep step between two groups of 4 waves (KG = 2), for
// grids that leave CUs idle.
//
// Loop.  Patch parts and weights go global -> LDS with buffer_load ... lds.
// Each step waits until the next step's weights are in LDS (a vmcnt count;
// loads retire in order), passes one barrier, issues the loads of a later
// stage and, at the first NPG taps, a part of the next chunk's patch, and
// reads the next half-step's fragments while the current one is multiplied.  Loads past
// the last chunk go out with an empty descriptor (zeros arrive), so that the
// count of loads in flight is the same at every step.
//
// Measured on MI355X (general kernel -> this one): on 128 CUs 16 images of
// 14x14x256 -> 256 16.8 -> 12.0 us, 28x28x128 -> 128 14.4 -> 10.7 us, two
// images of 56x56x256 -> 256 25.7 -> 16.4 us (450 TFLOP/s) and of
// 28x28x512 -> 512 25.3 -> 19.6 us; on 256 CUs 32 images of 28x28x512 -> 512
// 125 -> 99 us (1190 TFLOP/s) and of 56x56x256 -> 256 124-130 -> 110-115 us (by
// the data: 1030-1080 TFLOP/s).  By the counters no unit is full: on VGG-19 b8
// the LDS port moves 67 bytes per clock and CU, the matrix cores are busy 0.40
// of the time, and waves wait on dependencies (0.35) and to issue (0.35), which
// is block start, epilogue and the barrier of every step.  With one chunk of
// 64 channels the patch is used once and the general kernel's smaller blocks
// can be as fast (16 images of 56x56x64 -> 64 14.8 us there); the estimates of
// the dispatch keep those.
#include <algorithm>
#include <type_traits>

#include "common.hpp"
#include "conv_common.hpp"

namespace dstack {

struct HaloArgs {
  const bf16* x;
  const bf16* w;
  const float* scale;  // nullptr: 1
  const float* shift;  // nullptr: 0
  const bf16* res;     // nullptr: no residual
  bf16* y;
  float* partial;      // split-K workspace [splits][M][K]
  unsigned* counters;  // split-K: per-tile arrival counters (zero between launches)
  int N, H, W, C, K;
  int M;               // pixels
  int act;
  int chunks_per_split;  // 64-channel chunks per depth slice
  int tiles_n, tiles;
  int th, tw, tiles_h, tiles_w;  // tw > 0: output tiles of th x tw pixels; tw = 0: BM consecutive pixels
  int pw;                        // patch row width (W, or tw + 2)
  FastDiv div_w, div_h, div_tn, div_tw, div_pw, div_tiw, div_tih;
};

constexpr int HALO_TAPS = 9;

// Loads in flight, younger than the weights of step u + 1, when the wait of
// step u is reached (a step reads the first fragments of the next one); a
// patch part is issued before the weights at each of the first NPG steps.
template <int STAGES, int WL, int NPG>
constexpr int halo_wait(int u) {
  int n = (STAGES - 3) * WL;
  for (int v = u - (STAGES - 3); v < u; ++v) n += (v + HALO_TAPS) % HALO_TAPS < NPG ? 1 : 0;
  return n;
}

// bytes of LDS: the weight ring and two patches, later the staged output tile
template <int BN, int BM, int NW, int KG, int STAGES, int NPG, bool SPLIT>
constexpr int halo_lds() {
  const int loop = STAGES * BN * 128 + 2 * NPG * NW * 8 * 128;
  const int out = KG == 1 && !SPLIT ? BM * BN * 2 : KG * BM * BN * 4;
  return loop > out ? loop : out;
}

template <int BN, int BM, int WN, int WM, int KG, int STAGES, int NPG, bool SPLIT>
__global__ __launch_bounds__(64 * WN * WM * KG) void conv_halo_kernel(HaloArgs a) {
  constexpr int NW = WN * WM * KG;
  constexpr int NT = 64 * NW;
  constexpr int WSTAGE = BN * 128;           // bytes of one weight stage
  constexpr int WL = BN / 8 / NW;            // weight wave-loads per wave per step
  constexpr int PR = NPG * NW * 8;           // patch rows (the last one stays zero)
  constexpr int PB = PR * 128;               // bytes of one patch buffer
  constexpr int TN = BN / WN / 16, TM = BM / WM / 16;
  constexpr int NKS = 2 / KG;                // 32-deep halves of a 64-channel chunk per wave
  static_assert(BN % (8 * NW) == 0 && WL >= 1, "weight stage");
  static_assert(NPG <= 11 - STAGES && STAGES >= 4, "the last patch part must land before the next chunk");
  static_assert(KG == 1 || KG == 2, "depth groups");
  constexpr int LDS_BYTES = halo_lds<BN, BM, NW, KG, STAGES, NPG, SPLIT>();
  static_assert(LDS_BYTES <= 160 * 1024, "LDS of a CU");
  __shared__ __attribute__((aligned(1024))) unsigned char hlds[LDS_BYTES];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int kg = wave / (WN * WM), wg = wave - kg * (WN * WM);
  const int wn = wg % WN, wm = wg / WN;
  int tile;
  {
    const int L = blockIdx.x, q = a.tiles >> 3, r = a.tiles & 7, x = L & 7, i = L >> 3;
    tile = x * q + min(x, r) + i;
  }
  const int tm_idx = a.div_tn.div(tile);
  const int n0 = (tile - tm_idx * a.tiles_n) * BN;
  const int m0 = tm_idx * BM;
  int img = 0, h0 = 0, w0 = 0;
  if (a.tw > 0) {
    const int t2 = a.div_tiw.div(tm_idx);
    w0 = (tm_idx - t2 * a.tiles_w) * a.tw;
    img = a.div_tih.div(t2);
    h0 = (t2 - img * a.tiles_h) * a.th;
  }

  const int Kg = HALO_TAPS * a.C;
  const i32x4 wrs = make_rsrc(a.w, (unsigned)((long)a.K * Kg * 2));
  const i32x4 xrs = make_rsrc(a.x, (unsigned)((long)a.M * a.C * 2));
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);
  const unsigned lds0 = __builtin_amdgcn_readfirstlane(lds_address(hlds));
  const unsigned patch0 = lds0 + STAGES * WSTAGE;

  const int nchunk_total = a.C >> 6;
  int ck0 = 0, ck1 = nchunk_total;
  if (SPLIT) {
    ck0 = blockIdx.z * a.chunks_per_split;
    ck1 = min(nchunk_total, ck0 + a.chunks_per_split);
  }

  // lane's part of every wave-load: 16-byte chunk (lane % 8) of row lane / 8 of an 8-row group
  const int rin = lane >> 3;
  unsigned woff[WL];
#pragma unroll
  for (int j = 0; j < WL; ++j) {
    const int r = 8 * (wave * WL + j) + rin;
    const int c = (lane & 7) ^ ((r >> 1) & 7);
    const int n = n0 + r;
    woff[j] = n < a.K ? (unsigned)(((long)n * Kg + c * 8) * 2) : OOB;
  }
  unsigned poff[NPG];  // input byte offset of the lane's patch rows at channel 0
#pragma unroll
  for (int q = 0; q < NPG; ++q) {
    const int i = 8 * (q * NW + wave) + rin;
    const int c = (lane & 7) ^ ((i >> 1) & 7);
    if (a.tw > 0) {
      const int py = a.div_pw.div(i), px = i - py * a.pw;
      const int hi = h0 - 1 + py, wi = w0 - 1 + px;
      const bool ok = (unsigned)hi < (unsigned)a.H && (unsigned)wi < (unsigned)a.W && py < a.th + 2 && i < PR - 1;
      poff[q] = ok ? (unsigned)((((long)(img * a.H + hi) * a.W + wi) * a.C + c * 8) * 2) : OOB;
    } else {
      const int p = m0 - a.W - 1 + i;
      poff[q] = (unsigned)p < (unsigned)a.M && i < PR - 1 ? (unsigned)(((long)p * a.C + c * 8) * 2) : OOB;
    }
  }
  // the weights at tap `tap` of chunk ck
  auto issue_w = [&](int ck, int tap, int slot) __attribute__((always_inline)) {
    i32x4 rs = wrs;
    rs[2] = ck < ck1 ? rs[2] : 0;  // past the end: nothing is in range, zeros arrive
    const unsigned d = (unsigned)((tap * a.C + ck * 64) * 2);
    unsigned wv[WL];
#pragma unroll
    for (int j = 0; j < WL; ++j) wv[j] = woff[j] + d;
    load_group<WL>(rs, wv, lds0 + slot * WSTAGE + wave_u * WL * 1024);
  };
  auto issue_p = [&](int ck, int q, int buf) __attribute__((always_inline)) {
    i32x4 rs = xrs;
    rs[2] = ck < ck1 ? rs[2] : 0;
    unsigned pv[1] = {poff[q] + (unsigned)(ck * 128)};
    load_group<1>(rs, pv, patch0 + buf * PB + (q * NW + wave_u) * 1024);
  };

  // prologue: the first chunk's patch, then STAGES - 1 weight stages
#pragma unroll
  for (int q = 0; q < NPG; ++q) issue_p(ck0, q, 0);
#pragma unroll
  for (int s = 0; s < STAGES - 1; ++s) issue_w(ck0, s, s);

  // the wave's pixel fragments: patch row of the lane's pixel at tap (0, 0)
  // and the taps inside the image (a tile of th x tw pixels has zeros around
  // it in the patch itself, and reads every tap)
  const int cq = (lane >> 4) + 4 * kg;
  int prow[TM];
  unsigned pmask[TM];
#pragma unroll
  for (int j = 0; j < TM; ++j) {
    const int pl = wm * (BM / WM) + j * 16 + (lane & 15);
    if (a.tw > 0) {
      const int ty = a.div_tw.div(pl), tx = pl - ty * a.tw;
      prow[j] = ty * a.pw + tx;
      pmask[j] = ty < a.th ? 0x1ffu : 0u;
    } else {
      const int m = m0 + pl;
      const int t = a.div_w.div(m), wo = m - t * a.W, ho = t - a.div_h.div(t) * a.H;
      prow[j] = pl;
      const unsigned cols = (wo > 0 ? 1u : 0u) | 2u | (wo < a.W - 1 ? 4u : 0u);
      pmask[j] = m < a.M ? (ho > 0 ? cols : 0u) | cols << 3 | (ho < a.H - 1 ? cols << 6 : 0u) : 0u;
    }
  }
  // output pixel of local pixel pl (-1: none)
  auto out_pixel = [&](int pl) __attribute__((always_inline)) {
    if (a.tw > 0) {
      const int ty = a.div_tw.div(pl), tx = pl - ty * a.tw;
      const int h = h0 + ty, w = w0 + tx;
      return ty < a.th && h < a.H && w < a.W ? (img * a.H + h) * a.W + w : -1;
    }
    return m0 + pl < a.M ? m0 + pl : -1;
  };
  // The lane's residual values.  A 64 x 128 tile loads them before its loop,
  // where a round trip after it (0.8 us) is a tenth of a layer of one chunk: 91
  // shapes with a residual take 0.957 of their time so, and from 1.26 to 1.07
  // at most of the general kernel's.  The first steps' waits cover these loads,
  // which are issued behind the first stages.  The large tile has no registers
  // to spare for them and its 20 us of loop gain nothing (1.00, up to 1.05).
  constexpr bool RES_EARLY = KG == 1 && !SPLIT && TM * TN <= 8;
  bf16x4 resv[RES_EARLY ? TM : 1][TN] = {};
  auto load_res = [&](int j, bf16x4 (&r)[TN]) __attribute__((always_inline)) {
    const int px = max(out_pixel(wm * (BM / WM) + j * 16 + (lane & 15)), 0);
#pragma unroll
    for (int i = 0; i < TN; ++i) {
      const int c = min(n0 + wn * (BN / WN) + i * 16 + (lane >> 4) * 4, a.K - 4);
      r[i] = *reinterpret_cast<const bf16x4*>(a.res + ((long)px * a.K + c));
    }
  };
  if constexpr (RES_EARLY)
    if (a.res) {
#pragma unroll
      for (int j = 0; j < TM; ++j) load_res(j, resv[j]);
    }
  const int arow = wn * (BN / WN) + (lane & 15);
  const int aaddr = arow * 128 + ((cq ^ ((arow >> 1) & 7)) << 4);

  f32x4 acc[TN][TM];
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int j = 0; j < TM; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  // fragments: `f` of the half-step being multiplied, `g` of the next one
  bf16x8 fa[TN], fb[TM], ga[TN], gb[TM];
  int pa[TM];  // LDS offsets of the pixel fragments at the current tap
  auto at_tap = [&](int tap) __attribute__((always_inline)) {
    const int off = tap / 3 * a.pw + tap % 3;
#pragma unroll
    for (int j = 0; j < TM; ++j) {
      const int row = (pmask[j] >> tap) & 1 ? prow[j] + off : PR - 1;
      pa[j] = row * 128 + ((cq ^ ((row >> 1) & 7)) << 4);
    }
  };
  auto read = [&](bf16x8 (&ra)[TN], bf16x8 (&rb)[TM], int slot, int buf, int ks) __attribute__((always_inline)) {
    const unsigned char* sb = hlds + slot * WSTAGE + (aaddr ^ (ks * 64));
    const unsigned char* pb = hlds + STAGES * WSTAGE + buf * PB;
#pragma unroll
    for (int i = 0; i < TN; ++i) ra[i] = *reinterpret_cast<const bf16x8*>(sb + i * 2048);
#pragma unroll
    for (int j = 0; j < TM; ++j) rb[j] = *reinterpret_cast<const bf16x8*>(pb + (pa[j] ^ (ks * 64)));
  };
  // products of one half-step; the reads of the next one are spread over them
  auto mul = [&](const bf16x8 (&ra)[TN], const bf16x8 (&rb)[TM]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
      for (int j = 0; j < TM; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ra[i], rb[j], acc[i][j], 0, 0, 0);
#pragma unroll
    for (int q = 0; q < TN + TM; ++q) {
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, TN * TM / (TN + TM), 0);
    }
  };
  wait_vmcnt<(STAGES - 2) * WL>();
  __syncthreads();
  at_tap(0);
  read(fa, fb, 0, 0, 0);
  int rd = 0, wr = STAGES - 1, par = 0;
  for (int ck = ck0; ck < ck1; ++ck) {
    auto step = [&](auto uc) __attribute__((always_inline)) {
      constexpr int u = decltype(uc)::value, u1 = (u + 1) % HALO_TAPS, un = u + STAGES - 1;
      wait_vmcnt<halo_wait<STAGES, WL, NPG>(u)>();
      __syncthreads();
      if (u < NPG) issue_p(ck + 1, u < NPG ? u : 0, par ^ 1);
      issue_w(ck + un / HALO_TAPS, un % HALO_TAPS, wr);
      const int rn = rd + 1 == STAGES ? 0 : rd + 1;
      const int buf1 = u == HALO_TAPS - 1 ? par ^ 1 : par;
      if (NKS == 2) {
        read(ga, gb, rd, par, 1);
        mul(fa, fb);
        at_tap(u1);
        read(fa, fb, rn, buf1, 0);
        mul(ga, gb);
      } else {
        at_tap(u1);
        read(ga, gb, rn, buf1, 0);
        mul(fa, fb);
#pragma unroll
        for (int i = 0; i < TN; ++i) fa[i] = ga[i];
#pragma unroll
        for (int j = 0; j < TM; ++j) fb[j] = gb[j];
      }
      rd = rn;
      wr = wr + 1 == STAGES ? 0 : wr + 1;
    };
    step(std::integral_constant<int, 0>{});
    step(std::integral_constant<int, 1>{});
    step(std::integral_constant<int, 2>{});
    step(std::integral_constant<int, 3>{});
    step(std::integral_constant<int, 4>{});
    step(std::integral_constant<int, 5>{});
    step(std::integral_constant<int, 6>{});
    step(std::integral_constant<int, 7>{});
    step(std::integral_constant<int, 8>{});
    par ^= 1;
  }

  const float hi = a.act == ACT_RELU6 ? 6.0f : INFINITY;
  // f(act) with the activation chosen once: none, a clamp to [0, hi] (ReLU:
  // hi = inf), GELU or tanh
  auto with_act = [&](auto f) __attribute__((always_inline)) {
    if (a.act == ACT_NONE)
      f([](float v) { return v; });
    else if (a.act == ACT_GELU)
      f([](float v) { return gelu_erf(v); });
    else if (a.act == ACT_TANH)
      f([](float v) { return tanhf(v); });
    else
      f([hi](float v) { return fminf(fmaxf(v, 0.0f), hi); });
  };

  if (KG == 1 && !SPLIT) {
    // every lane finishes its 4 channels of a pixel in registers; the bf16
    // tile then goes through LDS ([pixel][channel] rows of 16-byte units
    // swizzled by the pixel) to leave in 16-byte pieces of whole rows
    f32x4 sc[TN], sh[TN];
#pragma unroll
    for (int i = 0; i < TN; ++i) {
      const int cc = min(n0 + wn * (BN / WN) + i * 16 + (lane >> 4) * 4, a.K - 4);
      sc[i] = a.scale ? *reinterpret_cast<const f32x4*>(a.scale + cc) : f32x4{1.f, 1.f, 1.f, 1.f};
      sh[i] = a.shift ? *reinterpret_cast<const f32x4*>(a.shift + cc) : f32x4{0.f, 0.f, 0.f, 0.f};
    }
    constexpr int UPR = BN / 8;  // 16-byte units per pixel row
    auto unit = [](int pl, int u) { return pl * UPR + (u ^ (UPR == 16 ? pl & 15 : (pl >> 1) & 7)); };
    static_assert(UPR == 16 || UPR == 8, "row swizzle");
    wait_vmcnt<0>();
    __syncthreads();  // all waves are done with the stages, no load is in flight
    with_act([&](auto act) __attribute__((always_inline)) {
#pragma unroll
      for (int j = 0; j < TM; ++j) {
        const int pl = wm * (BM / WM) + j * 16 + (lane & 15);
        bf16x4 (&r4)[TN] = resv[RES_EARLY ? j : 0];
        if constexpr (!RES_EARLY)
          if (a.res) load_res(j, r4);
#pragma unroll
        for (int i = 0; i < TN; ++i) {
          const int c = wn * (BN / WN) + i * 16 + (lane >> 4) * 4;
          bf16x4 o;
#pragma unroll
          for (int e = 0; e < 4; ++e) o[e] = (bf16)act(acc[i][j][e] * sc[i][e] + sh[i][e] + (float)r4[i][e]);
          *reinterpret_cast<bf16x4*>(hlds + unit(pl, c >> 3) * 16 + (c & 4) * 2) = o;
        }
      }
    });
    __syncthreads();
    constexpr int RS = NT / UPR, RPT = BM / RS;
    static_assert(NT % UPR == 0 && BM % RS == 0, "output thread mapping");
    const int u = tid % UPR, ch = n0 + u * 8, p0 = tid / UPR;
    if (ch >= a.K) return;
    uint4 v[RPT];
#pragma unroll
    for (int k = 0; k < RPT; ++k) v[k] = *reinterpret_cast<const uint4*>(hlds + unit(p0 + k * RS, u) * 16);
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
      const int px = out_pixel(p0 + k * RS);
      if (px >= 0) __builtin_memcpy(a.y + ((long)px * a.K + ch), &v[k], 16);  // (any alignment: one store)
    }
    return;
  }

  // fp32 tiles of the depth groups side by side in LDS, summed as they are
  // read back: thread -> 4 channels of ROWS_PT pixels
  constexpr int G = BN / 4;
  constexpr int RSTEP = NT / G;
  constexpr int ROWS_PT = BM / RSTEP;
  static_assert(NT % G == 0 && BM % RSTEP == 0 && G >= 8, "epilogue thread mapping");
  const int cl = (tid % G) * 4;
  const int ch0 = n0 + cl;
  const int pl0 = tid / G;
  const int chc = min(ch0, a.K - 4);
  const f32x4 sc = a.scale ? *reinterpret_cast<const f32x4*>(a.scale + chc) : f32x4{1.f, 1.f, 1.f, 1.f};
  const f32x4 sh = a.shift ? *reinterpret_cast<const f32x4*>(a.shift + chc) : f32x4{0.f, 0.f, 0.f, 0.f};
  wait_vmcnt<0>();
  __syncthreads();
  float* ct = reinterpret_cast<float*>(hlds);
  auto cidx = [](int pl, int cl) { return pl * BN + ((((cl >> 2) ^ (pl & 7))) << 2); };
#pragma unroll
  for (int i = 0; i < TN; ++i) {
    const int c = wn * (BN / WN) + i * 16 + (lane >> 4) * 4;
#pragma unroll
    for (int j = 0; j < TM; ++j) {
      const int pl = wm * (BM / WM) + j * 16 + (lane & 15);
      *reinterpret_cast<f32x4*>(ct + kg * BN * BM + cidx(pl, c)) = acc[i][j];
    }
  }
  __syncthreads();
  f32x4 t[ROWS_PT];
  int px[ROWS_PT];
#pragma unroll
  for (int k = 0; k < ROWS_PT; ++k) {
    const int e = cidx(pl0 + k * RSTEP, cl);
    t[k] = *reinterpret_cast<const f32x4*>(ct + e);
#pragma unroll
    for (int g = 1; g < KG; ++g) t[k] += *reinterpret_cast<const f32x4*>(ct + g * BN * BM + e);
    px[k] = out_pixel(pl0 + k * RSTEP);
  }
  if (SPLIT) {
    const unsigned slice_bytes = (unsigned)a.M * (unsigned)a.K * 4u;
    const __amdgpu_buffer_rsrc_t pr =
        __builtin_amdgcn_make_buffer_rsrc(a.partial, (short)0, (int)(slice_bytes * gridDim.z), 0x00020000);
    if (ch0 < a.K) {
#pragma unroll
      for (int k = 0; k < ROWS_PT; ++k)
        if (px[k] >= 0)
          __builtin_amdgcn_raw_buffer_store_b128(
              t[k], pr, (int)(blockIdx.z * slice_bytes + ((unsigned)px[k] * a.K + ch0) * 4u), 0, CPOL_SC1);
    }
    wait_vmcnt<0>();
    __syncthreads();
    int* flag = reinterpret_cast<int*>(hlds);
    if (tid == 0)
      *flag = (int)__hip_atomic_fetch_add(a.counters + tile, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (*flag != (int)gridDim.z - 1) return;
    if (tid == 0) __hip_atomic_store(a.counters + tile, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (ch0 >= a.K) return;
    const int S = gridDim.z;
    constexpr int ZC = ROWS_PT >= 16 ? 1 : 16 / ROWS_PT;
    for (int z0 = 0; z0 < S; z0 += ZC) {
      f32x4 q[ZC][ROWS_PT];
#pragma unroll
      for (int c = 0; c < ZC; ++c) {
        const unsigned z = (unsigned)min(z0 + c, S - 1);
#pragma unroll
        for (int k = 0; k < ROWS_PT; ++k)
          q[c][k] = __builtin_amdgcn_raw_buffer_load_b128(
              pr, (int)(z * slice_bytes + ((unsigned)max(px[k], 0) * a.K + ch0) * 4u), 0, CPOL_SC1);
      }
#pragma unroll
      for (int c = 0; c < ZC; ++c)
        if (z0 + c < S)
#pragma unroll
          for (int k = 0; k < ROWS_PT; ++k) t[k] = z0 + c == 0 ? q[c][k] : t[k] + q[c][k];
    }
  }
  if (ch0 >= a.K) return;
  bf16x4 rv[ROWS_PT];
#pragma unroll
  for (int k = 0; k < ROWS_PT; ++k)
    rv[k] = a.res ? *reinterpret_cast<const bf16x4*>(a.res + ((long)max(px[k], 0) * a.K + ch0)) : bf16x4{};
  with_act([&](auto act) __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < ROWS_PT; ++k) {
      if (px[k] < 0) continue;
      float v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = act(t[k][e] * sc[e] + sh[e] + (float)rv[k][e]);
      store_out4(a.y, false, (long)px[k] * a.K + ch0, v);
    }
  });
}

// ---- dispatch ----

// Tile shapes: channels x pixels, ring stages, patch rows (less the zero row), blocks that
// share a CU, whether it has a depth split, and the estimate of a block's time
// in us: fixed part and per 64-deep step, with one block on the CU and with two
// (fit to MI355X timings of 9, 18, 36 and 72 steps).  Only the 64 x 64 tile
// splits: the 64 x 128 tile's reduction needs 492 registers (one wave per SIMD
// and a spill), so that its blocks did not share a CU (7 images of 50x50x768 ->
// 176 on 240 CUs in two slices 106 us, unsplit in the general kernel 65; over
// 60 shapes that took it the present choice takes 0.80 of its time).
struct HaloTile {
  int bn, bm, stages, rows, per_cu;
  bool split;
  double fix1, step1, fix2, step2;
};
static constexpr HaloTile kHalo[] = {
    {64, 128, 4, 191, 2, false, 3.25, 0.217, 4.15, 0.333},
    {64, 64, 6, 127, 2, true, 3.0, 0.152, 3.2, 0.232},
    {128, 256, 4, 383, 1, false, 6.9, 0.574, 0, 0},
};
constexpr int kHaloTiles = 3, kHaloLarge = 2, kHaloRest = 0;

template <int BN, int BM, int WN, int WM, int KG, int STAGES, int NPG, bool CAN_SPLIT>
static void halo_go(const HaloArgs& a, int splits, hipStream_t st, hipEvent_t e0, hipEvent_t e1) {
  const dim3 grid(a.tiles, 1, splits);
  constexpr int NT = 64 * WN * WM * KG;
  if constexpr (CAN_SPLIT) {
    if (splits > 1) {
      launch_k(conv_halo_kernel<BN, BM, WN, WM, KG, STAGES, NPG, true>, grid, NT, st, e0, e1, a);
      return;
    }
  }
  launch_k(conv_halo_kernel<BN, BM, WN, WM, KG, STAGES, NPG, false>, grid, NT, st, e0, e1, a);
}

// th x tw tiles (or tw = 0: consecutive pixels) for tile shape t with the
// fewest blocks over one image size; false if none fits its patch.
static bool halo_shape(const HaloTile& t, int n, int H, int W, int* th, int* tw, long* tiles) {
  *tiles = 0;
  if (t.bm + 2 * W + 2 <= t.rows) {
    *th = *tw = 0;
    *tiles = ((long)n * H * W + t.bm - 1) / t.bm;
  }
  // the tile rows of 16 pixels fill a fragment; the others cover widths that 16 does not divide
  for (int w : {16, 32, 28, 14, 8}) {
    const int h = t.bm / w;
    if (w > W || h < 1 || (h + 2) * (w + 2) > t.rows) continue;
    const long k = (long)n * ceil_div(H, h) * ceil_div(W, w);
    if (*tiles == 0 || k < *tiles) {
      *tiles = k;
      *th = h;
      *tw = w;
    }
  }
  return *tiles > 0;
}

// Estimated time of a launch.  Tiles that fill a CU's LDS are counted on whole
// groups of 32 CUs: blocks are dealt evenly to the 4 shader engines of each of
// the 8 XCDs, so with other CU counts an engine's last block waits for a CU
// while another engine's stays idle (78 such blocks took two rounds on 80 CUs).
static int halo_cus(const HaloTile& t, int n_cu) { return t.per_cu == 1 && n_cu >= 32 ? n_cu / 32 * 32 : n_cu; }
static double halo_cost(const HaloTile& t, long blocks, int steps, int n_cu) {
  const double one = t.fix1 + steps * t.step1, two = t.fix2 + steps * t.step2;
  n_cu = halo_cus(t, n_cu);
  if (t.per_cu == 1) return (double)((blocks + n_cu - 1) / n_cu) * one;
  const long full = blocks / (2L * n_cu), rem = blocks - full * 2L * n_cu;
  return full * two + (rem > n_cu ? two : rem > 0 ? one : 0.0);
}

bool halo_plan(int N, int H, int W, int C, int K, int n_cu, bool can_split, size_t split_bytes, HaloPlan* out) {
  const int chunks = C / 64;
  const long M = (long)N * H * W;
  // never more slices than the allocation-free entry point's scratch holds
  split_bytes = std::min(split_bytes, CONV_SCRATCH_BYTES - SPLITK_TILE_COUNTERS * sizeof(unsigned));
  out->cost = 1e30;
  for (int i = 0; i < kHaloTiles; ++i) {
    const HaloTile& t = kHalo[i];
    int th, tw;
    long tm;
    if ((t.bn > 64 && K <= 64) || !halo_shape(t, N, H, W, &th, &tw, &tm)) continue;
    const long tiles = tm * ceil_div(K, t.bn);
    if (tiles > 0x7fffffffL) continue;
    for (int sp = 1; sp <= 8; sp *= 2) {
      if (sp > 1 && (!t.split || !can_split || sp > chunks || (size_t)sp * M * K * sizeof(float) > split_bytes ||
                     tiles > SPLITK_TILE_COUNTERS))
        break;
      const int per = ceil_div(chunks, sp), s = ceil_div(chunks, per);
      double c = halo_cost(t, tiles * s, per * HALO_TAPS, n_cu);
      // the last block's read-back costs half of what the general kernel's
      // estimate says (one image of 7x7x512: 8.2 us in 8 slices, 9.1 in 4)
      if (s > 1) c += CONV_SLICE_WRITE_US + 0.5 * CONV_SLICE_READ_US * s * (t.bn * t.bm) / 8192.0;
      if (c < out->cost * 0.97) *out = HaloPlan{i, th, tw, s, per, N, -1, 0, 0, c};
    }
  }
  // Whole rounds, then the rest: the largest tile on as many images as fill
  // every CU the same number of times, the remaining images in 64 x 128 tiles
  // that share all CUs, when the partly filled last round costs more than a
  // second launch (about 1.3 us).
  {
    const HaloTile& t = kHalo[kHaloLarge];
    const HaloTile& r = kHalo[kHaloRest];
    int th, tw, th2, tw2;
    long tm, tm2;
    if (K > 64 && N > 1 && halo_shape(t, N, H, W, &th, &tw, &tm)) {
      const int tn = ceil_div(K, t.bn);
      const int cus = halo_cus(t, n_cu);
      const long rounds = tm * tn / cus;
      int n1 = (int)std::min<long>(N, rounds * cus / tn * t.bm / ((long)H * W));
      if (rounds > 0 && n1 > 0 && n1 < N && halo_shape(t, n1, H, W, &th, &tw, &tm) &&
          halo_shape(r, N - n1, H, W, &th2, &tw2, &tm2)) {
        const int steps = chunks * HALO_TAPS;
        const double c = halo_cost(t, tm * tn, steps, n_cu) + 1.3 + halo_cost(r, tm2 * ceil_div(K, r.bn), steps, n_cu);
        if (c < out->cost * 0.97) *out = HaloPlan{kHaloLarge, th, tw, 1, chunks, n1, kHaloRest, th2, tw2, c};
      }
    }
  }
  return out->cost < 1e29;
}

void halo_tile(const HaloPlan& p, int* bn, int* bm, int* stages) {
  *bn = kHalo[p.tile].bn;
  *bm = kHalo[p.tile].bm;
  *stages = kHalo[p.tile].stages;
}

void launch_halo(const bf16* x, int N, int H, int W, int C, const bf16* w, int K, const float* scale,
                 const float* shift, const bf16* res, int act, bf16* y, const HaloPlan& p, float* splitk_ws,
                 unsigned* tile_counters, hipStream_t st) {
  auto part = [&](int tile, int th, int tw, int n0, int n, hipEvent_t e0, hipEvent_t e1) {
    const HaloTile& t = kHalo[tile];
    HaloArgs a{};
    const size_t px = (size_t)n0 * H * W;
    a.x = x + px * C; a.w = w; a.scale = scale; a.shift = shift; a.res = res ? res + px * K : nullptr;
    a.y = y + px * K;
    a.N = n; a.H = H; a.W = W; a.C = C; a.K = K; a.M = n * H * W; a.act = act;
    a.chunks_per_split = p.chunks_per_split;
    if (p.splits > 1) {
      a.partial = splitk_ws;
      a.counters = tile_counters;
    }
    a.th = th; a.tw = tw;
    a.tiles_n = ceil_div(K, t.bn);
    a.tiles_h = tw > 0 ? ceil_div(H, th) : 1;
    a.tiles_w = tw > 0 ? ceil_div(W, tw) : 1;
    a.tiles = (tw > 0 ? n * a.tiles_h * a.tiles_w : ceil_div(a.M, t.bm)) * a.tiles_n;
    a.pw = tw > 0 ? tw + 2 : W;
    a.div_w = FastDiv::make(W);
    a.div_h = FastDiv::make(H);
    a.div_tn = FastDiv::make(a.tiles_n);
    a.div_tw = FastDiv::make(tw > 0 ? tw : 1);
    a.div_pw = FastDiv::make(a.pw);
    a.div_tiw = FastDiv::make(a.tiles_w);
    a.div_tih = FastDiv::make(a.tiles_h);
    switch (tile) {
      case 0: halo_go<64, 128, 1, 4, 1, 4, 6, false>(a, p.splits, st, e0, e1); break;
      case 1: halo_go<64, 64, 1, 4, 2, 6, 2, true>(a, p.splits, st, e0, e1); break;
      default: halo_go<128, 256, 2, 4, 1, 4, 6, false>(a, p.splits, st, e0, e1); break;
    }
  };
  const DispatchEvents& de = dispatch_events();
  const bool two = p.n_main < N;
  part(p.tile, p.th, p.tw, 0, p.n_main, de.start, two ? nullptr : de.stop);
  if (two) part(p.rest_tile, p.rest_th, p.rest_tw, p.n_main, N - p.n_main, nullptr, de.stop);
}

}  // namespace dstack
