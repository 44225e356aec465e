// The LSTM recurrence of a whole sequence in one launch (Sec. 4.1's
// memory-bound example):
//   gates[b][g*H + j] = gx[t][b][g*H + j] + sum_k W_hh[g*H + j][k] * h(t-1)[b][k]
//   c = f*c + i*g~, h = o*tanh(c)            (gate order i, f, g, o; h = c = 0 before t = 0)
//
// One launch per step (kernels_seq.hip) reads all of W_hh every step and is
// bound by those loads and by the launch: 5.9 us a step for B = 32, H = 1024
// on 128 CUs.  Here W_hh is read once, into registers: the blocks of a group
// (one batch slice of at most 16 items) each own RT row tiles, i.e. 4 RT
// hidden units with their four gates, and the 8 waves of a block split the
// depth.  What remains is a chain of T exchanges of h between the blocks,
// about 1 us each through device-scope memory, and the cell update: 3.2 us a
// step on 128 CUs (layer 322 -> 182 us with its input projection; B = 4
// 253 -> 132, B = 1 242 -> 165; H = 256, B = 8 on 48 CUs 181 -> 94).  The cell
// is the step path's: its divisions and its tanhf cost 0.25 and 0.2 us of a
// step against v_rcp and 1 - 2 / (1 + e^2x) (159 us), which were up to 6 ulp
// off.
//
// Exchange.  Two slots of h in bf16, laid out [k/8][item][8], written with
// device-scope 16-byte stores (narrower ones cost up to 0.7 us a step more)
// and polled with device-scope loads until every value has arrived: |h| <= 1,
// so bit 14 of its bf16 is free and carries the parity of t / 2, which tells
// a slot's new values from those of two steps ago; a NaN travels as 0x3fff,
// above every |h|.  No flags and no barrier between blocks: a block writes
// h(t+2) into the slot of h(t) only after it has seen all of h(t+1), which
// its group computed after reading all of h(t).
//
// Waiting.  The blocks of a group must run at the same time, so the plan asks
// for no more blocks than the dispatcher places at once (lstm_seq_blocks).
// If others hold the CUs all the same (recurrences released together on
// CUs that they share, each resident in part), every wait is bounded: it gives
// up after `limit` or when another wave did, and the blocks that run compute
// the sequence from its start as shared work, without the others (lstm_shared).
// Measured with 50 steps, B = 32, H = 1024: two layers released together on 16
// slots each, 8 of them shared, 0.39 ms (0.46 by one launch per step), four on
// the same 16 slots, of which three give up, 2.1 ms (0.86); shared work alone
// takes 0.55 ms, 10 us a step.
#include <algorithm>

#include "common.hpp"
#include "conv_common.hpp"

namespace dstack {

namespace {

constexpr int LS_WAVES = 8;
constexpr int LS_THREADS = 64 * LS_WAVES;
constexpr int LS_TS = 1024 + 128;  // LDS bytes of one 16 x 16 partial tile (padded: adjacent tiles, other banks)

// control words: [1] a wait gave up; from these on, steps done and taken of each block's rows and items
constexpr int LS_DONE = 64, LS_TAKEN = LS_DONE + 256;

struct LstmSeqArgs {
  const float* gx;   // [T][B][4H]
  const bf16* whh;   // [4H][H]
  bf16* h;           // [T][B][H]
  float* hf;         // [T][B][H] or null
  float* c;          // [B][H]: cell state (shared work only)
  unsigned* xch;     // exchanged h, two slots of groups * H * bg bf16
  unsigned short* hp;  // h of shared work, two slots of [H/32][B][32] bf16
  unsigned* ctl;     // control words
  int T, B, H, groups, bg, blocks;
  long limit;        // ticks (10 ns) a wait may last
};

__device__ __forceinline__ unsigned bf16_bits(bf16 v) { return (unsigned)__builtin_bit_cast(unsigned short, v); }

// The recurrence as shared work, when a wait gave up.  A unit is one step of
// one block's rows and items; two words of each block's unit count the steps
// taken and done.  The current step is the least that is done of any unit; a
// block takes its own unit of it (whose weights its XCD's L2 holds), else one
// that nobody took: that of a block which does not run.  Every wait ends,
// however few of the launch's blocks run: a taken unit belongs to a block that
// runs, and a running block takes what is left of the current step before it
// waits.  Blocks that start later join.  h goes through hp and c through memory
// (device scope, complete before the unit counts as done); what blocks that
// have not yet noticed write to h and hf meanwhile are the same values up to
// summation order.
template <int RT, int KSW>
__device__ void lstm_shared(const LstmSeqArgs& a, unsigned char* red, int* pick) {
  constexpr int CELLS = RT * 4 * 16;
  const int tid = threadIdx.x, lane = tid & 63, quad = lane >> 4, col = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // scalar: products past the depth are branched around
  const int H = a.H, B = a.B, nks = H >> 5, k0 = wave * KSW, own = blockIdx.x;
  const int slot_elems = B * H;
  const __amdgpu_buffer_rsrc_t hr = __builtin_amdgcn_make_buffer_rsrc(a.hp, (short)0, slot_elems * 4, 0x00020000);
  unsigned* const done = a.ctl + LS_DONE;
  unsigned* const taken = a.ctl + LS_TAKEN;
  const int cb = (tid >> 3) & 15, cu = (tid >> 7) * 8 + (tid & 7);  // the thread's cell, as in the kernel
  auto wave_min = [](int v) __attribute__((always_inline)) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v = min(v, __shfl_xor(v, o, 64));
    return __builtin_amdgcn_readfirstlane(v);
  };
  // The loops' control is scalar and barriers enclose the divergent branches of
  // this one: were one joined with another across the back edge, its lanes
  // would circle alone, barriers included, and never end.
  for (;;) {
    __syncthreads();  // partial sums, flags and pick have been read
    if (wave == 0) {
      int t, unit = -1;
      for (;;) {
        int least = a.T, key = 0x7fffffff;
        unsigned tk[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int m = lane + 64 * j;
          const bool in = m < a.blocks;
          tk[j] = in ? __hip_atomic_load(taken + m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : ~0u;
          if (in) least = min(least, (int)__hip_atomic_load(done + m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        }
        t = wave_min(least);
        if (t >= a.T) break;
        // the own unit first, the others in an order that differs from block to block
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int m = lane + 64 * j;
          if (tk[j] == (unsigned)t) key = min(key, m == own ? m : ((m * 97 + own * 61 & 255) + 1) << 8 | m);
        }
        key = wave_min(key);
        if (key == 0x7fffffff) continue;  // all taken: wait
        unsigned was = (unsigned)t;
        if (lane == 0)
          __hip_atomic_compare_exchange_strong(taken + (key & 255), &was, (unsigned)t + 1, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT);
        if (__builtin_amdgcn_readfirstlane((int)was) == t) {
          unit = key & 255;
          break;
        }
      }
      *(volatile int*)&pick[0] = t;
      *(volatile int*)&pick[1] = unit;
    }
    __syncthreads();
    const int t = __builtin_amdgcn_readfirstlane(*(volatile int*)&pick[0]);
    const int unit = __builtin_amdgcn_readfirstlane(*(volatile int*)&pick[1]);
    if (unit < 0) return;
    const int grp = unit % a.groups, rt0 = unit / a.groups * RT;
    const int b0 = grp * a.bg, nb = min(a.bg, B - b0);
    const int cj = 4 * rt0 + cu, item = b0 + cb;
    const bool mine = tid < CELLS && cb < nb;
    const long cell = (long)item * H + cj;
    float g4[4], cst = 0.f;
#pragma unroll
    for (int g = 0; g < 4; ++g) g4[g] = mine ? a.gx[((long)t * B + item) * 4 * H + g * H + cj] : 0.f;
    if (t > 0) {
      const int slot = ((t - 1) & 1) * slot_elems * 2, b = b0 + min(col, nb - 1);
      if (mine) cst = __hip_atomic_load(a.c + cell, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      bf16x8 x[KSW];
#pragma unroll
      for (int s = 0; s < KSW; ++s)
        if (k0 + s < nks)
          x[s] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(
                                                hr, (((k0 + s) * B + b) * 32 + quad * 8) * 2, slot, CPOL_SC1));
#pragma unroll
      for (int i = 0; i < RT; ++i) {
        const bf16* wr = a.whh + (long)((col >> 2) * H + 4 * (rt0 + i) + (col & 3)) * H + k0 * 32 + quad * 8;
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < KSW; ++s)
          if (k0 + s < nks)
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*reinterpret_cast<const bf16x8*>(wr + s * 32), x[s], acc, 0, 0, 0);
#pragma unroll
        for (int u = 0; u < 4; ++u)
          *reinterpret_cast<float*>(red + (wave * RT + i) * LS_TS + (u * 16 + col) * 16 + quad * 4) = acc[u];
      }
    }
    __syncthreads();
    if (mine) {
      if (t > 0) {
        f32x4 v[LS_WAVES];
#pragma unroll
        for (int q = 0; q < LS_WAVES; ++q)
          v[q] = *reinterpret_cast<const f32x4*>(red + (q * RT + (cu >> 2)) * LS_TS + ((cu & 3) * 16 + cb) * 16);
        const f32x4 sum = ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
#pragma unroll
        for (int g = 0; g < 4; ++g) g4[g] += sum[g];
      }
      float hn;
      lstm_cell(g4, cst, hn);
      const bf16 hb = (bf16)hn;
      __hip_atomic_store(a.hp + (t & 1) * slot_elems + ((cj >> 5) * B + item) * 32 + (cj & 31),
                         __builtin_bit_cast(unsigned short, hb), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(a.c + cell, cst, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const long o = (long)t * B * H + cell;
      a.h[o] = hb;
      if (a.hf) a.hf[o] = hn;
    }
    wait_vmcnt<0>();  // the wave's stores have reached device scope
    __syncthreads();
    if (wave == 0) __hip_atomic_store(done + unit, (unsigned)(t + 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

template <int RT, int KSW>
__global__ __launch_bounds__(LS_THREADS, RT <= 4 && RT * KSW <= 8 ? 4 : 2) void lstm_seq_kernel(LstmSeqArgs a) {
  constexpr int TS = LS_TS;
  constexpr int BUF = LS_WAVES * RT * TS;   // partial sums of one step
  constexpr int CELLS = RT * 4 * 16;
  static_assert(CELLS <= LS_THREADS, "one thread per cell");
  __shared__ __attribute__((aligned(16))) unsigned char red[2 * BUF];
  // by step modulo 3: items whose h(t-1) holds a NaN (bits 0..15), and
  // whether a wave gave up waiting (bit 16)
  __shared__ int flags[3];
  const int tid = threadIdx.x, lane = tid & 63, quad = lane >> 4, col = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // scalar: products past the depth are branched around
  const int H = a.H, nks = H >> 5, tiles = H >> 2;
  const int grp = blockIdx.x % a.groups, rank = blockIdx.x / a.groups;
  const int b0 = grp * a.bg, nb = min(a.bg, a.B - b0);  // the group's batch items
  const int rt0 = rank * RT;
  const int k0 = wave * KSW;  // first depth step of the wave
  const unsigned slot_elems = (unsigned)(a.groups * H * a.bg);
  const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(a.xch, (short)0, (int)(slot_elems * 4u), 0x00020000);
  if (tid < 3) flags[tid] = 0;

  // W_hh fragments of the wave, kept for the whole sequence
  bf16x8 w[RT][KSW];
#pragma unroll
  for (int i = 0; i < RT; ++i)
#pragma unroll
    for (int s = 0; s < KSW; ++s) {
      const int rt = rt0 + i, ks = k0 + s;
      w[i][s] = rt < tiles && ks < nks
                    ? *reinterpret_cast<const bf16x8*>(a.whh + (long)((col >> 2) * H + 4 * rt + (col & 3)) * H + ks * 32 + quad * 8)
                    : bf16x8{};
    }

  // the thread's cell: unit cj, item cb
  const int cb = (tid >> 3) & 15, cu = (tid >> 7) * 8 + (tid & 7);
  const int cj = 4 * rt0 + cu;
  const int cl = (cu >> 2) * TS + ((cu & 3) * 16 + cb) * 16;
  const bool mine = tid < CELLS && cj < H && cb < nb;
  float cst = 0.f, gxv[4];
  const float* gxp = a.gx + (long)(b0 + cb) * 4 * H + cj;
#pragma unroll
  for (int g = 0; g < 4; ++g) gxv[g] = mine ? gxp[g * H] : 0.f;
  // byte offset of the lane's 8 values of depth step k0 (columns past the group's items read its last one)
  const int xoff = (int)((unsigned)(grp * H * a.bg + ((k0 * 4 + quad) * a.bg + max(0, min(col, nb - 1))) * 8) * 2u);
  const int kstep_bytes = 4 * a.bg * 16;
  const int woff = (int)((unsigned)(grp * H * a.bg + ((cj >> 3) * a.bg + cb) * 8 + (cj & 7)) * 2u);

  __syncthreads();
  bool dead = false, gave_up = false;
  for (int t = 0, t3 = 0; t < a.T; ++t, t3 = t3 == 2 ? 0 : t3 + 1) {
    unsigned char* rb = red + (t & 1) * BUF;
    if (t > 0) {
      const unsigned phase = ((t - 1) >> 1) & 1 ? 0x40004000u : 0u;
      const int slot = (int)(((t - 1) & 1) * slot_elems * 2u);
      typedef unsigned x_t[KSW][4];
      x_t x;
      auto load = [&](x_t& d) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < KSW; ++s)
          if (k0 + s < nks) {
            const uint4 v = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(xr, xoff + s * kstep_bytes, slot, CPOL_SC1));
            d[s][0] = v.x; d[s][1] = v.y; d[s][2] = v.z; d[s][3] = v.w;
          }
      };
      auto ready = [&](const x_t& d) __attribute__((always_inline)) {
        unsigned bad = 0;
#pragma unroll
        for (int s = 0; s < KSW; ++s)
          if (k0 + s < nks)
#pragma unroll
            for (int e = 0; e < 4; ++e) bad |= d[s][e] ^ phase;
        return __ballot((bad & 0x40004000u) != 0) == 0;
      };
      long t0 = 0;
      for (int spin = 0;; ++spin) {
        load(x);
        if (ready(x)) break;
        if ((spin & 15) == 15 || a.limit < 0) {  // bounded: give up after `limit`, or when another wave did
          const long now = (long)__builtin_amdgcn_s_memrealtime();
          if (spin <= 15) t0 = now;
          if (now - t0 > a.limit || __hip_atomic_load(a.ctl + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
            dead = true;
            break;
          }
        }
      }
      if (dead && lane == 0) {
        __hip_atomic_store(a.ctl + 1, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        atomicOr(&flags[t3], 1 << 16);
      }
      f32x4 acc[RT];
#pragma unroll
      for (int i = 0; i < RT; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < KSW; ++s) {
        if (k0 + s >= nks) break;
        const uint4 hv = {x[s][0] & 0xbfffbfffu, x[s][1] & 0xbfffbfffu, x[s][2] & 0xbfffbfffu, x[s][3] & 0xbfffbfffu};
        const bf16x8 hb = __builtin_bit_cast(bf16x8, hv);
#pragma unroll
        for (int i = 0; i < RT; ++i) acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[i][s], hb, acc[i], 0, 0, 0);
      }
      // NaN codes (0x3fff: above every |h| <= 1) in the lane's item
      typedef __attribute__((__vector_size__(2 * sizeof(unsigned short)))) unsigned short u16x2;
      unsigned top = 0;
#pragma unroll
      for (int s = 0; s < KSW; ++s)
        if (k0 + s < nks)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const u16x2 p = __builtin_bit_cast(u16x2, x[s][e] & 0x3fff3fffu), q = __builtin_bit_cast(u16x2, top);
            top = __builtin_bit_cast(unsigned, __builtin_elementwise_max(p, q));
          }
      if ((top & 0xffffu) == 0x3fffu || (top >> 16) == 0x3fffu) atomicOr(&flags[t3], 1 << col);
      // [unit][item][gate]: lane (gate quad, item col) holds the tile's 4 units
#pragma unroll
      for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int u = 0; u < 4; ++u)
          *reinterpret_cast<float*>(rb + (wave * RT + i) * TS + (u * 16 + col) * 16 + quad * 4) = acc[i][u];
    }
    __syncthreads();
    const int flag = __builtin_amdgcn_readfirstlane(*(volatile int*)&flags[t3]);
    float g4[4] = {gxv[0], gxv[1], gxv[2], gxv[3]};
    if (t > 0 && wave * 64 < CELLS) {
      f32x4 v[LS_WAVES];
#pragma unroll
      for (int k = 0; k < LS_WAVES; ++k) v[k] = *reinterpret_cast<const f32x4*>(rb + k * RT * TS + cl);
      const f32x4 sum = ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
#pragma unroll
      for (int g = 0; g < 4; ++g) g4[g] += sum[g];
    }
    if (flag >> 16) {  // the same in all waves: written before the barrier
      gave_up = true;
      break;
    }
    // read by all before this step's barrier, set again after the next one's
    if (tid == 0) *(volatile int*)&flags[t3 == 0 ? 2 : t3 - 1] = 0;
    if (wave * 64 >= CELLS) continue;  // wave-uniform: no cells
    if ((flag >> cb) & 1) g4[0] = g4[1] = g4[2] = g4[3] = __builtin_nanf("");
    float hn;
    lstm_cell(g4, cst, hn);
    const bf16 hb = (bf16)hn;
    if (t + 1 < a.T) {
      // the 8 units of an item (8 consecutive lanes) leave as one 16-byte store
      const unsigned code = (hn != hn ? 0x3fffu : bf16_bits(hb)) | ((t >> 1) & 1 ? 0x4000u : 0u);
      const unsigned c1 = __builtin_amdgcn_mov_dpp(code, 0xb1, 0xf, 0xf, true);  // lane ^ 1
      const unsigned lo = lane & 1 ? c1 | code << 16 : code | c1 << 16;
      const unsigned c2 = __builtin_amdgcn_mov_dpp(lo, 0x4e, 0xf, 0xf, true);    // lane ^ 2
      const unsigned q0 = lane & 2 ? c2 : lo, q1 = lane & 2 ? lo : c2;
      const unsigned r0 = __builtin_amdgcn_mov_dpp(q0, 0x141, 0xf, 0xf, true);   // 7 - lane of 8
      const unsigned r1 = __builtin_amdgcn_mov_dpp(q1, 0x141, 0xf, 0xf, true);
      typedef __attribute__((__vector_size__(4 * sizeof(unsigned)))) unsigned u32x4;
      if (mine && (lane & 7) == 0)
        __builtin_amdgcn_raw_buffer_store_b128((u32x4{q0, q1, r0, r1}), xr, woff, (int)((t & 1) * slot_elems * 2u), CPOL_SC1);
    }
    if (mine) {
      if (t + 1 < a.T) {
        gxp += (long)a.B * 4 * H;
#pragma unroll
        for (int g = 0; g < 4; ++g) gxv[g] = gxp[g * H];
      }
      const long o = ((long)t * a.B + b0 + cb) * H + cj;
      a.h[o] = hb;
      if (a.hf) a.hf[o] = hn;
    }
  }
  if (gave_up) lstm_shared<RT, KSW>(a, red, flags);
}

// marks both slots as not yet written (bit 14 set: the parity of t / 2 = 1), clears the control words
static_assert(LSTM_SEQ_CTL_BYTES == (LS_TAKEN + 256) * 4, "a plan has at most 256 blocks");
__global__ __launch_bounds__(256) void lstm_seq_clear_kernel(unsigned* xch, int n, unsigned* ctl) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) xch[i] = 0x40004000u;
  if (i < LSTM_SEQ_CTL_BYTES / 4) ctl[i] = 0u;
}

}  // namespace

template <int KSW>
static void lstm_seq_rt(const LstmSeqArgs& a, int rt, hipStream_t st) {
  const dim3 grid(a.blocks), blk(LS_THREADS);
  if (KSW == 8 || rt == 2)
    launch(lstm_seq_kernel<2, KSW>, grid, blk, 0, st, a);
  else if constexpr (KSW <= 4) {
    if (rt == 4)
      launch(lstm_seq_kernel<4, KSW>, grid, blk, 0, st, a);
    else
      launch(lstm_seq_kernel<8, KSW>, grid, blk, 0, st, a);
  }
}

// Blocks (one per CU) that CUs hold at once: `mask` is a stream's CU mask of
// 256 bits, byte j the CUs of slot j, one on each XCD; null: the first n_cu / 8
// slots.  Blocks go round robin to the XCDs and, in each, to the shader
// engines that have CUs in the mask (slot j is on engine j % 4), whichever
// engine still has room: with engines of unequal size the smallest fills first
// and holds the others up (10 blocks per XCD on engines of 3, 3, 2 and 2 CUs
// took two rounds).  A mask with a part of a slot gives the XCDs different
// engines, which this does not count: no room.
static int lstm_seq_blocks(int n_cu, const uint32_t* mask) {
  int per[4] = {0, 0, 0, 0};
  for (int slot = 0; slot < 32; ++slot) {
    const uint32_t cus = mask ? (mask[slot / 4] >> (8 * (slot % 4))) & 0xffu : slot < n_cu / 8 ? 0xffu : 0u;
    if (cus != 0 && cus != 0xffu) return 0;
    if (cus) ++per[slot % 4];
  }
  int least = 0, engines = 0;
  for (int c : per)
    if (c > 0) {
      least = engines == 0 ? c : std::min(least, c);
      ++engines;
    }
  return 8 * engines * least;
}

// The fewest row tiles per block that the CUs allow (more CUs on a group's
// rows means fewer products and partial sums on each: RT = 2 / 4 / 8 takes
// 2.9 / 3.0 / 3.4 us a step for 16 items, H = 1024), groups of at most 16
// items (one MFMA column tile).  A block's weights must fit its registers:
// RT * (depth steps per wave) <= 32.  Sequences of fewer than 4 steps and
// partitions that cannot hold a group stay with one launch per step.
bool lstm_seq_plan(int T, int B, int H, int n_cu, const uint32_t* mask, LstmSeqPlan* out) {
  if (T < 4) return false;
  const int tiles = H / 4, groups = (B + 15) / 16;
  int ksw = 1;
  while (ksw * LS_WAVES * 32 < H) ksw *= 2;
  if (ksw > 8) return false;
  const int room = lstm_seq_blocks(n_cu, mask);
  for (int rt = 2; rt <= (ksw == 8 ? 2 : 8); rt *= 2) {
    const int blocks = groups * ((tiles + rt - 1) / rt);
    if (blocks > room) continue;
    *out = LstmSeqPlan{groups, rt, blocks};
    return true;
  }
  return false;
}

bool lstm_seq_plan(int T, int B, int H, int n_cu, hipStream_t st, LstmSeqPlan* out) {
  uint32_t words[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  int bits = 0;
  if (st && hipExtStreamGetCUMask(st, 8, words) == hipSuccess)
    for (uint32_t w : words) bits += __builtin_popcount(w);
  else if (st)
    (void)hipGetLastError();
  // (a launch planned for other CUs than the stream's: as for consecutive slots)
  return lstm_seq_plan(T, B, H, n_cu, bits == n_cu ? words : static_cast<const uint32_t*>(nullptr), out);
}

size_t lstm_seq_exchange_bytes(int B, int H, const LstmSeqPlan& p) {
  return (size_t)2 * p.groups * ((B + p.groups - 1) / p.groups) * H * 2;
}

dstack_status launch_lstm_seq(const float* gx, const bf16* whh, bf16* h, float* hf, float* c, void* exchange,
                              bf16* hp, unsigned* ctl, int T, int B, int H, const LstmSeqPlan& p, long limit, hipStream_t st) {
  DS_CHECK(B >= 1 && B <= 32 && H % 32 == 0 && H >= 32 && H <= 2048, DSTACK_E_UNSUPPORTED, "lstm: bad shape");
  LstmSeqArgs a{gx, whh, h, hf, c, static_cast<unsigned*>(exchange), reinterpret_cast<unsigned short*>(hp), ctl,
                T, B, H, p.groups,
                (B + p.groups - 1) / p.groups, p.blocks, limit};
  const int words = (int)(lstm_seq_exchange_bytes(B, H, p) / 4);
  launch(lstm_seq_clear_kernel, dim3((std::max(words, (int)LSTM_SEQ_CTL_BYTES / 4) + 255) / 256), dim3(256), 0, st, a.xch,
         words, ctl);
  DS_HIP(hipGetLastError());
  const int ksw = (H / 32 + LS_WAVES - 1) / LS_WAVES;
  if (ksw <= 1)
    lstm_seq_rt<1>(a, p.row_tiles, st);
  else if (ksw <= 2)
    lstm_seq_rt<2>(a, p.row_tiles, st);
  else if (ksw <= 4)
    lstm_seq_rt<4>(a, p.row_tiles, st);
  else
    lstm_seq_rt<8>(a, p.row_tiles, st);
  DS_HIP(hipGetLastError());
  return DSTACK_OK;
}

}  // namespace dstack
