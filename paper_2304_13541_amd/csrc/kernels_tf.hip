// Transformer kernels of the BERT encoder (Sec. 4.4's transformer workload):
// token embedding + layer norm, layer norm, and the multi-head
// self-attention core.  The encoder's matrix products run on the
// implicit-GEMM convolution kernel as 1x1 convolutions (bias, residual,
// GELU and tanh in its epilogue).
//
// Layer norm (alone and after the embedding sum): one wave per token row, the
// row's values in registers as 16-byte pieces, mean and (biased) variance by
// fp32 wave reductions, output bf16.  No barrier; gamma and beta are loaded
// with the row, so a wave waits for memory once, which with the launch is
// what bounds it.  Rows of a width that is no multiple of 8 or of tensors
// that are not 16-byte aligned take one 256-thread block each, with element
// loads and block reductions.  Measured on MI355X, wave against block: 320
// rows of 768 2.8 us against 3.5 (with the embedding sum 2.9 against 3.8),
// 2048 rows 3.4 against 5.0, 20000 rows 11.7 against 36.5.
//
// Attention: one block per (head, sequence), one wave per 16 queries of the
// sequence's T <= 48 tokens (64 dims per head), everything in registers on the
// matrix cores.  Scores as S^T = K Q^T (v_mfma_f32_16x16x32_bf16: bf16
// products, fp32 sums): a lane then holds four keys 4 * (lane / 16) + i of
// each 16-key tile for the query lane % 16, the softmax is a reduction over
// its own values and the four lanes of that query, and the fp32 weights are
// already the B operand of O^T = V^T P^T on v_mfma_f32_16x16x4_f32 (step i of
// a tile takes key 4 * quad + i; the sum over keys has no order to keep).  The
// weights so stay fp32.  Row m of dim tile t is dim 4 m + t: a lane reads four
// consecutive dims of a key (8 bytes) and ends with 16 consecutive dims of
// its query, two 16-byte stores.  All of a wave's loads are issued at its
// start: the kernel is bound by that one latency and the launch.  Measured on
// MI355X, 16 sequences of 20 tokens, 12 heads: 3.3 us against 8.6 for the
// same sums as fp32 vector arithmetic from LDS (three barriers, scalar
// loads); 32 sequences of 48 tokens 28.3 -> 6.1 us.
#include <initializer_list>

#include "common.hpp"

namespace dstack {

namespace {

constexpr int LN_MAX_PER_THREAD = 8;  // rows of up to 2048 values
constexpr int ATT_DH = 64;            // head width
constexpr int ATT_MAX_T = 48;         // tokens per sequence

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// sum over the 256-thread block (every thread gets the total)
__device__ __forceinline__ float block_sum(float v, float* red) {
  v = wave_sum(v);
  const int wave = threadIdx.x >> 6;
  __syncthreads();  // red may still be read from the previous call
  if ((threadIdx.x & 63) == 0) red[wave] = v;
  __syncthreads();
  return red[0] + red[1] + red[2] + red[3];
}

// normalise the thread's values of one row of H and write them as bf16
__device__ __forceinline__ void ln_row(float (&v)[LN_MAX_PER_THREAD], int H, const float* gamma, const float* beta,
                                       float eps, bf16* y, float* red) {
  float s = 0.f;
#pragma unroll
  for (int j = 0; j < LN_MAX_PER_THREAD; ++j)
    if ((int)threadIdx.x + j * 256 < H) s += v[j];
  const float mean = block_sum(s, red) / (float)H;
  float q = 0.f;
#pragma unroll
  for (int j = 0; j < LN_MAX_PER_THREAD; ++j)
    if ((int)threadIdx.x + j * 256 < H) q += (v[j] - mean) * (v[j] - mean);
  const float inv = rsqrtf(block_sum(q, red) / (float)H + eps);
#pragma unroll
  for (int j = 0; j < LN_MAX_PER_THREAD; ++j) {
    const int c = threadIdx.x + j * 256;
    if (c < H) {
      float o = (v[j] - mean) * inv;
      if (gamma) o *= gamma[c];
      if (beta) o += beta[c];
      y[c] = (bf16)o;
    }
  }
}

__global__ __launch_bounds__(256) void embed_ln_kernel(const int* __restrict__ ids, int T, int vocab,
                                                       const bf16* __restrict__ we, const bf16* __restrict__ pe,
                                                       const bf16* __restrict__ te, int H, const float* gamma,
                                                       const float* beta, float eps, bf16* __restrict__ y) {
  __shared__ float red[4];
  const int row = blockIdx.x;
  const int t = row % T;
  const int id = min(max(ids[row], 0), vocab - 1);  // ids outside the vocabulary read its last row
  float v[LN_MAX_PER_THREAD];
#pragma unroll
  for (int j = 0; j < LN_MAX_PER_THREAD; ++j) {
    const int c = threadIdx.x + j * 256;
    v[j] = c < H ? (float)we[(long)id * H + c] + (float)pe[(long)t * H + c] + (float)te[c] : 0.f;
  }
  ln_row(v, H, gamma, beta, eps, y + (long)row * H, red);
}

__global__ __launch_bounds__(256) void layernorm_kernel(const bf16* __restrict__ x, int H, const float* gamma,
                                                        const float* beta, float eps, bf16* __restrict__ y) {
  __shared__ float red[4];
  const long row = blockIdx.x;
  float v[LN_MAX_PER_THREAD];
#pragma unroll
  for (int j = 0; j < LN_MAX_PER_THREAD; ++j) {
    const int c = threadIdx.x + j * 256;
    v[j] = c < H ? (float)x[row * H + c] : 0.f;
  }
  ln_row(v, H, gamma, beta, eps, y + row * H, red);
}

// One row of H = 8 * units values by one wave: lane l holds the 16-byte
// pieces l, l + 64, ... (at most J).
template <int J>
__device__ __forceinline__ void ln_wave(float (&v)[J][8], int units, const float* gamma, const float* beta, float eps,
                                        bf16* y) {
  const int lane = threadIdx.x & 63;
  f32x4 g[J][2], b[J][2];
#pragma unroll
  for (int j = 0; j < J; ++j)
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int c = min(lane + 64 * j, units - 1) * 8 + 4 * e;
      g[j][e] = gamma ? *reinterpret_cast<const f32x4*>(gamma + c) : f32x4{1.f, 1.f, 1.f, 1.f};
      b[j][e] = beta ? *reinterpret_cast<const f32x4*>(beta + c) : f32x4{0.f, 0.f, 0.f, 0.f};
    }
  const float H = (float)(8 * units);
  float s = 0.f;
#pragma unroll
  for (int j = 0; j < J; ++j)
    if (lane + 64 * j < units)
#pragma unroll
      for (int e = 0; e < 8; ++e) s += v[j][e];
  const float mean = wave_sum(s) / H;
  float q = 0.f;
#pragma unroll
  for (int j = 0; j < J; ++j)
    if (lane + 64 * j < units)
#pragma unroll
      for (int e = 0; e < 8; ++e) q += (v[j][e] - mean) * (v[j][e] - mean);
  const float inv = rsqrtf(wave_sum(q) / H + eps);
#pragma unroll
  for (int j = 0; j < J; ++j) {
    if (lane + 64 * j >= units) continue;
    bf16x8 o;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      float n = (v[j][e] - mean) * inv;
      if (gamma) n *= g[j][e >> 2][e & 3];
      if (beta) n += b[j][e >> 2][e & 3];
      o[e] = (bf16)n;
    }
    *reinterpret_cast<bf16x8*>(y + (lane + 64 * j) * 8) = o;
  }
}

template <int J>
__global__ __launch_bounds__(64) void layernorm_wave_kernel(const bf16* __restrict__ x, int units,
                                                            const float* gamma, const float* beta, float eps,
                                                            bf16* __restrict__ y) {
  const long row = (long)blockIdx.x * 8 * units;
  float v[J][8];
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const bf16x8 t = *reinterpret_cast<const bf16x8*>(x + row + min((int)threadIdx.x + 64 * j, units - 1) * 8);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[j][e] = (float)t[e];
  }
  ln_wave<J>(v, units, gamma, beta, eps, y + row);
}

template <int J>
__global__ __launch_bounds__(64) void embed_ln_wave_kernel(const int* __restrict__ ids, int T, int vocab,
                                                           const bf16* __restrict__ we, const bf16* __restrict__ pe,
                                                           const bf16* __restrict__ te, int units,
                                                           const float* gamma, const float* beta, float eps,
                                                           bf16* __restrict__ y) {
  const int row = blockIdx.x, H = 8 * units;
  const int id = min(max(ids[row], 0), vocab - 1);  // ids outside the vocabulary read its last row
  float v[J][8];
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const int c = min((int)threadIdx.x + 64 * j, units - 1) * 8;
    const bf16x8 w = *reinterpret_cast<const bf16x8*>(we + (long)id * H + c);
    const bf16x8 p = *reinterpret_cast<const bf16x8*>(pe + (long)(row % T) * H + c);
    const bf16x8 t = *reinterpret_cast<const bf16x8*>(te + c);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[j][e] = (float)w[e] + (float)p[e] + (float)t[e];
  }
  ln_wave<J>(v, units, gamma, beta, eps, y + (long)row * H);
}

// whole 16-byte pieces everywhere (null pointers count as aligned)
bool ln_vector(int H, std::initializer_list<const void*> ptrs) {
  uintptr_t bits = 0;
  for (const void* p : ptrs) bits |= (uintptr_t)p;
  return H % 8 == 0 && (bits & 15) == 0;
}

// N consecutive bf16 values; one load where the tensor is 16-byte aligned
template <int N, bool ALIGNED, typename V>
__device__ __forceinline__ V load_bf16(const bf16* p) {
  V v;
  if (ALIGNED) {
    v = *reinterpret_cast<const V*>(p);
  } else {
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = p[i];
  }
  return v;
}

// NT = ceil(T / 16) waves and key tiles
template <int NT, bool ALIGNED>
__global__ __launch_bounds__(64 * NT) void attention_kernel(const bf16* __restrict__ qkv, int T, int width,
                                                            bf16* __restrict__ out) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, col = lane & 15, quad = lane >> 4;
  const long tok0 = (long)blockIdx.y * T;
  const bf16* base = qkv + tok0 * 3 * width + blockIdx.x * ATT_DH;
  const int query = wave * 16 + col;
  bf16x8 qf[2], kf[NT][2];
  bf16x4 vf[NT][4];
  auto row = [&](int t) { return base + (long)min(t, T - 1) * 3 * width; };  // rows past T are masked below
#pragma unroll
  for (int s = 0; s < 2; ++s) qf[s] = load_bf16<8, ALIGNED, bf16x8>(row(query) + s * 32 + quad * 8);
#pragma unroll
  for (int kt = 0; kt < NT; ++kt)
#pragma unroll
    for (int s = 0; s < 2; ++s)
      kf[kt][s] = load_bf16<8, ALIGNED, bf16x8>(row(kt * 16 + col) + width + s * 32 + quad * 8);
#pragma unroll
  for (int kt = 0; kt < NT; ++kt)
#pragma unroll
    for (int i = 0; i < 4; ++i)
      vf[kt][i] = load_bf16<4, ALIGNED, bf16x4>(row(kt * 16 + 4 * quad + i) + 2 * width + 4 * col);

  f32x4 p[NT];
  float mx = -INFINITY;
#pragma unroll
  for (int kt = 0; kt < NT; ++kt) {
    p[kt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < 2; ++s) p[kt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[kt][s], qf[s], p[kt], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      p[kt][i] *= 0.125f;  // 1 / sqrt(64)
      if (kt * 16 + 4 * quad + i < T) mx = fmaxf(mx, p[kt][i]);
    }
  }
  mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
  mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
  float sum = 0.f;
#pragma unroll
  for (int kt = 0; kt < NT; ++kt)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      p[kt][i] = kt * 16 + 4 * quad + i < T ? __expf(p[kt][i] - mx) : 0.f;
      sum += p[kt][i];
    }
  sum += __shfl_xor(sum, 16, 64);
  sum += __shfl_xor(sum, 32, 64);
  f32x4 o[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) o[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int kt = 0; kt < NT; ++kt)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bool live = kt * 16 + 4 * quad + i < T;
      const float w = p[kt][i] / sum;
#pragma unroll
      for (int t = 0; t < 4; ++t)
        o[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(live ? (float)vf[kt][i][t] : 0.f, w, o[t], 0, 0, 0);
    }
  if (query >= T) return;
  bf16* dst = out + (tok0 + query) * width + blockIdx.x * ATT_DH + 16 * quad;  // dim 16 * quad + 4 i + t
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    bf16x8 r;
#pragma unroll
    for (int j = 0; j < 8; ++j) r[j] = (bf16)o[j & 3][2 * u + (j >> 2)];
    if (ALIGNED) {
      *reinterpret_cast<bf16x8*>(dst + 8 * u) = r;
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) dst[8 * u + j] = r[j];
    }
  }
}

template <int NT>
void attention_launch(const bf16* qkv, int B, int T, int heads, bf16* out, hipStream_t st) {
  const dim3 grid((unsigned)heads, (unsigned)B);
  if ((((uintptr_t)qkv | (uintptr_t)out) & 15) == 0)  // rows are multiples of 128 bytes
    launch(attention_kernel<NT, true>, grid, dim3(64 * NT), 0, st, qkv, T, heads * ATT_DH, out);
  else
    launch(attention_kernel<NT, false>, grid, dim3(64 * NT), 0, st, qkv, T, heads * ATT_DH, out);
}

}  // namespace

dstack_status launch_embed_ln(const int* ids, int rows, int T, int vocab, const bf16* we, const bf16* pe,
                              const bf16* te, int H, const float* gamma, const float* beta, float eps, bf16* y,
                              hipStream_t st) {
  DS_CHECK(ids && we && pe && te && y, DSTACK_E_INVALID, "embed_ln: null pointer");
  DS_CHECK(rows > 0 && T > 0 && vocab > 0 && H > 0, DSTACK_E_INVALID, "embed_ln: bad shape");
  DS_CHECK(H <= 256 * LN_MAX_PER_THREAD, DSTACK_E_UNSUPPORTED, "embed_ln: width above 2048");
  const dim3 grid((unsigned)rows);
  if (!ln_vector(H, {we, pe, te, gamma, beta, y}))
    launch(embed_ln_kernel, grid, dim3(256), 0, st, ids, T, vocab, we, pe, te, H, gamma, beta, eps, y);
  else if (H <= 1024)
    launch(embed_ln_wave_kernel<2>, grid, dim3(64), 0, st, ids, T, vocab, we, pe, te, H / 8, gamma, beta, eps, y);
  else
    launch(embed_ln_wave_kernel<4>, grid, dim3(64), 0, st, ids, T, vocab, we, pe, te, H / 8, gamma, beta, eps, y);
  DS_HIP(hipGetLastError());
  return DSTACK_OK;
}

dstack_status launch_layernorm(const bf16* x, int rows, int H, const float* gamma, const float* beta, float eps,
                               bf16* y, hipStream_t st) {
  DS_CHECK(x && y, DSTACK_E_INVALID, "layernorm: null pointer");
  DS_CHECK(rows > 0 && H > 0, DSTACK_E_INVALID, "layernorm: bad shape");
  DS_CHECK(H <= 256 * LN_MAX_PER_THREAD, DSTACK_E_UNSUPPORTED, "layernorm: width above 2048");
  const dim3 grid((unsigned)rows);
  if (!ln_vector(H, {x, gamma, beta, y}))
    launch(layernorm_kernel, grid, dim3(256), 0, st, x, H, gamma, beta, eps, y);
  else if (H <= 1024)
    launch(layernorm_wave_kernel<2>, grid, dim3(64), 0, st, x, H / 8, gamma, beta, eps, y);
  else
    launch(layernorm_wave_kernel<4>, grid, dim3(64), 0, st, x, H / 8, gamma, beta, eps, y);
  DS_HIP(hipGetLastError());
  return DSTACK_OK;
}

dstack_status launch_attention(const bf16* qkv, int B, int T, int heads, int dh, bf16* out, hipStream_t st) {
  DS_CHECK(qkv && out, DSTACK_E_INVALID, "attention: null pointer");
  DS_CHECK(B > 0 && T > 0 && heads > 0, DSTACK_E_INVALID, "attention: bad shape");
  DS_CHECK(dh == ATT_DH && T <= ATT_MAX_T && heads <= 65535 && B <= 65535, DSTACK_E_UNSUPPORTED,
           "attention: head width 64 and at most 48 tokens");
  if (T <= 16)
    attention_launch<1>(qkv, B, T, heads, out, st);
  else if (T <= 32)
    attention_launch<2>(qkv, B, T, heads, out, st);
  else
    attention_launch<3>(qkv, B, T, heads, out, st);
  DS_HIP(hipGetLastError());
  return DSTACK_OK;
}

}  // namespace dstack
