// 3x3 stride-1 convolution of fp32 tensors (forward and data gradient) on the bf16 matrix core.
//
// Every fp32 operand a is taken apart into three bf16 numbers, a = h + m + l, each the nearest bf16 to what the ones
// before it leave: 8 + 8 + 8 significant bits, so nothing of a's 24 is lost.  A product is then six bf16 products
//   a*b = h*h' + (h*m' + m*h') + (m*m' + h*l' + l*h')      (what is left out is at most 2^-24 of |a*b|, 2^-27.5 in the mean)
// accumulated in fp32, small terms first.  v_mfma_f32_32x32x16_bf16 does 16 times the work of
// v_mfma_f32_32x32x2_f32 per cycle, so six of them take 6/16 of the time one fp32 product takes.
//
// Where that is not so, a workgroup computes its tile again on the fp32 matrix instruction: where a result is not finite
// (an infinity, or a finite value that rounds to one, leaves a NaN in the difference a - h and so in every output it
// reaches, and h*h' may overflow where a*b, within 0.8 % of the largest float, does not), and where it has staged an
// operand of so small a magnitude (below 2^-110; from 2^-103 up never) that its parts run out of bf16's bits.  A layer all of
// whose tiles are computed twice takes twice the time that the fp32 instruction takes on staged tiles (batch 128, all NaN:
// 64 ch 32x32 193 us, 128 ch 16x16 174, 256 ch 8x8 161, 512 ch 4x4 169; with one load in flight per wave 551, 524, 497, 925).
//
// What bounds this kernel is the staging: an operand element costs 5.5 vector instructions to take apart and 6 bytes of
// LDS.  So the input pixels of a tile are staged once per 64 channels and serve all nine taps: the tile is a range of
// BM consecutive pixels of the flattened [N*H*W], tap (r, s) of pixel m is pixel m + (r-1)*W + (s-1), so a range of
// BM + 2W + 2 pixels holds every tap, whatever H, W and the image boundaries are; a tap that falls off its image reads
// a row of zeros instead.
//
// Measured, us, fp32 instruction -> this kernel (forward | data gradient with its filter transpose):
//   batch 128: 64 ch 32x32  88 -> 68 | 94 -> 72    128 ch 16x16  83 -> 57 | 89 -> 61
//             256 ch  8x8   82 -> 50 | 89 -> 56    512 ch  4x4   90 -> 62 | 100 -> 72
//   batch  77: 64 ch 32x32  68 -> 49 | 74 -> 54    128 ch 16x16  65 -> 52 | 70 -> 56
//             256 ch  8x8   80 -> 59 | 87 -> 64    512 ch  4x4   89 -> 58 | 99 -> 65
// The matrix cores of the 256-channel forward kernel, batch 128, are busy 53 % of its cycles, at the 1.9 GHz that the shader
// holds under it (29 us; 23 at the nominal clock); the filter rows staged per tap cost 8 us of the rest, the fragment reads 4.
// Error against float64 over 27 to 4608 products per output: 1.6e-7 to 4.6e-7 (2-norm), the fp32 instruction's 2.5e-7 to
// 1.1e-6.
#include "conv_tile.h"

namespace resist {
namespace {

constexpr int kMaxW = 56;
constexpr int kBN = 64, kNT = 512, kBK = 64, kWGK = 4, kWGM = 2, kTN = 2;
constexpr int kPlane = kBK * 2;            // bytes of one part of a staged row
constexpr int kPitch = 3 * kPlane + 16;    // row pitch: rows 4 banks apart, conflict-free 16-byte reads of consecutive rows
constexpr int kStageB = kBN * kPitch;

// the three bf16 parts of four floats to their places in a staged row; returns what the first two leave, checked if CHECK
template <bool CHECK>
__device__ inline f32x4 store_split(char *row, f32x4 v, unsigned long long &missed) {
  f32x4 rest;
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    if (p == 2) {
      rest = v;
      if (CHECK) split_check(v, missed);
    }
    *reinterpret_cast<u32x2 *>(row + p * kPlane) = split_part(v);
  }
  return rest;
}

// 8 waves: 2 along the pixels, 4 sharing the reduction (wave slice k takes 16 of every 64 channels), so that a wave's
// tile is as large as the registers allow (BM/2 x 64): an operand fragment read from LDS feeds 2*TM or 2*TN products.
template <int BM, int MODE>
__global__ __launch_bounds__(kNT) void conv3_split_kernel(ArgsOf<MODE> a) {
  constexpr int WTM = BM / kWGM, TM = WTM / 32, NSUB = TM * kTN;
  constexpr int PA = (BM + 2 * kMaxW + 2 + 31) / 32, PB = kBN / 32;   // staging passes of 32 rows x 16 lanes
  constexpr int PX = PA * 32;                     // staged pixels; the row after them is zero
  constexpr int LDC = kBN + 8;
  constexpr size_t kOperand = 2 * kStageB + (size_t)(PX + 1) * kPitch;
  constexpr size_t kReduce = (size_t)kWGM * kWGK * NSUB * 4 * 64 * 16;
  constexpr size_t kTile = sizeof(float) * BM * LDC;
  constexpr size_t kBytes = kOperand > kReduce ? (kOperand > kTile ? kOperand : kTile) : (kReduce > kTile ? kReduce : kTile);
  __shared__ __attribute__((aligned(16))) char lds[kBytes];
  __shared__ int row_off[BM];
  char *const Bs = lds, *const Px = lds + 2 * kStageB;
  float (*Cs)[LDC] = reinterpret_cast<float (*)[LDC]>(lds);

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wk = wave & 3, wm = wave >> 2;
  const int lr = lane & 31, lg = lane >> 5;
  const int bid = xcd_contiguous(blockIdx.x, gridDim.x);
  const int tm = fdiv(bid, a.div_tn), tn = bid - tm * a.tiles_n;
  const int m0 = tm * BM, n0 = tn * kBN;
  const int W = a.IW, IC = a.IC, px = BM + 2 * W + 2;   // staged pixels: m0 - W - 1 .. m0 + BM + W
  const int cchunks = (IC + kBK - 1) / kBK;
  const int steps = 9 * cchunks;

  for (int r = tid; r < BM; r += kNT) row_off[r] = m0 + r < a.Mrows ? m0 + r : -1;

  // which taps of this lane's pixels lie inside their image, and where in LDS its operands start
  int valid[TM], abase[TM];
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int ml = wm * WTM + i * 32 + lr, m = m0 + ml;
    const int n = fdiv(m, a.div_plane), rem = m - n * (a.IH * W);
    const int h = fdiv(rem, a.div_w), w = rem - h * W;
    int v = 0;
#pragma unroll
    for (int t = 0; t < 9; ++t) {
      const int r = MODE == kBwd ? 2 - t / 3 : t / 3, s = MODE == kBwd ? 2 - t % 3 : t % 3;
      if ((unsigned)(h + r - 1) < (unsigned)a.IH && (unsigned)(w + s - 1) < (unsigned)W) v |= 1 << t;
    }
    valid[i] = m < a.Mrows ? v : 0;
    abase[i] = (ml + W + 1) * kPitch + wk * 32 + lg * 16;
  }
  const int zbase = PX * kPitch + wk * 32 + lg * 16;

  const __amdgpu_buffer_rsrc_t rin = make_rsrc(a.in, (unsigned)a.N * a.IH * W * IC * 4u);
  const __amdgpu_buffer_rsrc_t rwt = make_rsrc(a.wt, (unsigned)a.OC * 9u * IC * 4u);

  // ---- staging: 16 lanes (4 channels each) per row
  const int srow = tid >> 4, sch = (tid & 15) * 4;
  // filter stage of a set: where a thread stores its rows, where a lane fetches its fragments
  char *bdst[2] = {Bs + srow * kPitch + sch * 2, Bs + kStageB + srow * kPitch + sch * 2};
  const char *bsrc[2] = {Bs + lr * kPitch + wk * 32 + lg * 16, Bs + kStageB + lr * kPitch + wk * 32 + lg * 16};
  char *const pdst = Px + srow * kPitch + sch * 2;
  f32x4 rp[PA], rb[2][PB];
  unsigned long long missed = 0;   // operands that three parts do not hold
  unsigned boff[PB];
#pragma unroll
  for (int i = 0; i < PB; ++i) {
    const int oc = n0 + i * 32 + srow;
    boff[i] = oc < a.OC ? (unsigned)(oc * 9 * IC + sch) * 4u : kOOB;
  }
  // pixels before the first and past the last of the tensor come back as zeros (offsets wrap above the size)
  const unsigned poff = (unsigned)((m0 - W - 1 + srow) * IC + sch) * 4u;
  int pc = 0;                 // chunk of the pixels requested next
  auto request_pixels = [&]() {
    const bool ok = pc < cchunks && pc * kBK + sch < IC;
#pragma unroll
    for (int i = 0; i < PA; ++i) {
      unsigned o = ok && i * 32 + srow < px ? poff + (unsigned)(i * 32 * IC + pc * kBK) * 4u : kOOB;
      asm("" : "+v"(o));   // a selected offset; left alone, the compiler makes two loads behind a branch and waits for each
      rp[i] = buffer_load_16B(rin, o);
    }
    ++pc;
  };
  auto store_pixels = [&](int i) {
    if (i * 32 < px) store_split<true>(pdst + i * 32 * kPitch, rp[i], missed);   // uniform
  };
  int bt = 0, bc = 0;         // tap and chunk of the filter rows requested next
  auto request_filter = [&](int set) {
    const bool ok = bc < cchunks && bc * kBK + sch < IC;
    const unsigned d = (unsigned)(bt * IC + bc * kBK) * 4u;
#pragma unroll
    for (int i = 0; i < PB; ++i) rb[set][i] = buffer_load_16B(rwt, ok ? boff[i] + d : kOOB);
    const bool wrap = bt == 8;
    bt = wrap ? 0 : bt + 1;
    bc = wrap ? bc + 1 : bc;
  };
  // the rows of step t wait in register set t % 2 and go to LDS stage t % 2
  // 128-pixel tiles check the filter rows a group of products later, where nobody waits for it (128 ch 16x16, batch 128: 60.3 ->
  // 59.3 us; 64-pixel tiles, with half the products, 59.7 -> 61.5)
  constexpr bool kLater = TM == 2;
  f32x4 rest[PB];
  auto store_filter = [&](int set, int i) { rest[i] = store_split<!kLater>(bdst[set] + i * 32 * kPitch, rb[set][i], missed); };

  // ---- fragments: three parts of TM pixel tiles and kTN filter tiles.  A part is fetched for the next step as soon as
  // its last product of this step is issued; only the leading parts (index 0), which the last product of a step and the
  // first two of the next both use, have two register sets.
  f32x4 fa0[2][TM], fb0[2][kTN], fa[3][TM], fb[3][kTN];
  int ft = 0;                 // tap of the fragments fetched next
  int aat[TM];                // where that tap's pixel is
  auto aim = [&]() {
    const int r = ft / 3, s = ft - r * 3;
    const int d = ((r - 1) * W + s - 1) * (MODE == kBwd ? -kPitch : kPitch);
#pragma unroll
    for (int i = 0; i < TM; ++i) aat[i] = (valid[i] >> ft) & 1 ? abase[i] + d : zbase;
    ft = ft == 8 ? 0 : ft + 1;
  };
  auto fetch_a = [&](int set, int q) {
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const f32x4 v = *reinterpret_cast<const f32x4 *>(Px + aat[i] + q * kPlane);
      if (q == 0) fa0[set][i] = v;
      else fa[q][i] = v;
    }
  };
  auto fetch_b = [&](int set, int q) {
#pragma unroll
    for (int j = 0; j < kTN; ++j) {
      const f32x4 v = *reinterpret_cast<const f32x4 *>(bsrc[set] + j * 32 * kPitch + q * kPlane);
      if (q == 0) fb0[set][j] = v;
      else fb[q][j] = v;
    }
  };

  f32x16 acc[TM][kTN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < kTN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
  auto product = [&](int set, int pa, int pb, bool first = false) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < kTN; ++j)
        Elem<__bf16>::mma(acc[i][j], pa == 0 ? fa0[set][i] : fa[pa][i], pb == 0 ? fb0[set][j] : fb[pb][j]);
    if (first) {   // a product, half of the staging's arithmetic beside it, the other product
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x002, 14, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  auto lds_barrier = [&]() {
    __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
  };

  request_pixels();
  request_filter(0);
  request_filter(1);
  if (tid < 100) *reinterpret_cast<unsigned *>(Px + PX * kPitch + tid * 4) = 0;
#pragma unroll
  for (int i = 0; i < PA; ++i) store_pixels(i);
#pragma unroll
  for (int i = 0; i < PB; ++i) {
    store_filter(0, i);
    if (kLater) split_check(rest[i], missed);
  }
  request_filter(0);
  store_filter(1, 0);
  if (kLater) split_check(rest[0], missed);
  request_pixels();
  lds_barrier();
  aim();
#pragma unroll
  for (int q = 0; q < 3; ++q) { fetch_a(0, q); fetch_b(0, q); }
  __builtin_amdgcn_sched_barrier(0);

  // Step (chunk, tap), six groups of products, small terms first.  Beside them, spread so that neither the LDS nor the
  // vector unit sees a burst: the second half of the next step's filter rows goes to LDS and the rows three steps ahead
  // are requested (all workgroups walk the filter in step, so each row comes from beyond the L2 once per XCD and every
  // one of them waits for it); the barrier, after which the filter fragments of the next step are fetched; the first
  // half of the rows of the step after it.  The last step of a chunk also replaces the pixels: all fragments of this
  // chunk are in registers once its barrier is passed.  (The products stand outside the branches: inside, the
  // accumulators are copied.)
  static_assert(PB == 2, "filter rows per step");
  int tap = 0;
  auto step = [&](int set, int it) {
    const bool turn = tap == 8 && it + 1 < steps;   // uniform
    const int nx = set ^ 1;
    constexpr int H = (PA + 2) / 3;
    // turn, said by the tap that follows: the compiler joins branches on the same condition, and then copies the fragments that
    // the other side of it has just requested, a wait in every step (2 % of the kernel's time)
    auto replace = [&](int q) {
      if (ft == 1 && it + 1 < steps) {
#pragma unroll
        for (int i = q * H; i < (q + 1) * H && i < PA; ++i) store_pixels(i);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    aim();
    store_filter(nx, 1);
    product(set, 2, 0);
    if (!turn) fetch_a(nx, 2);
    request_filter(nx);
    product(set, 0, 2);
    lds_barrier();
    fetch_b(nx, 2);
    if (!turn) fetch_a(nx, 0);
    if (kLater) split_check(rest[1], missed);
    product(set, 1, 1);
    replace(0);
    fetch_b(nx, 0);
    product(set, 1, 0);
    replace(1);
    if (!turn) fetch_a(nx, 1);
    store_filter(set, 0);        // of step it + 2
    // (64-pixel data gradients: left alone, their wait for the filter rows comes before both products, 4 % of the time)
    product(set, 0, 1, MODE == kBwd && TM == 1);
    replace(2);
    fetch_b(nx, 1);
    if (turn) {
      request_pixels();
      lds_barrier();
#pragma unroll
      for (int q = 2; q >= 0; --q) fetch_a(nx, q);
    }
    if (kLater) split_check(rest[0], missed);
    product(set, 0, 0);
    tap = tap == 8 ? 0 : tap + 1;
  };
  // An odd number of steps starts with one on its own, after which the sets change places: a loop that could end between
  // its two steps makes the compiler wait for every load at its top.  (Behind the last step: rows nobody uses.)
  int it = 0;
  if (steps & 1) {
    step(0, 0);
    it = 1;
#pragma unroll
    for (int i = 0; i < TM; ++i) fa0[0][i] = fa0[1][i];
#pragma unroll
    for (int j = 0; j < kTN; ++j) fb0[0][j] = fb0[1][j];
#pragma unroll
    for (int i = 0; i < PB; ++i) { const f32x4 t = rb[0][i]; rb[0][i] = rb[1][i]; rb[1][i] = t; }
    char *const d = bdst[0]; bdst[0] = bdst[1]; bdst[1] = d;
    const char *const f = bsrc[0]; bsrc[0] = bsrc[1]; bsrc[1] = f;
    __builtin_amdgcn_sched_barrier(0);
  }
  do {
    step(0, it);
    step(1, it + 1);
    it += 2;
  } while (it < steps);

  conv_epilogue<float, BM, kBN, kNT, MODE>(a, Cs, row_off, tm, n0, [&]() {
    // the four slices of a wave tile are added in slice order; wave slice k finishes the k-th quarter of it
    f32x4 *const red = reinterpret_cast<f32x4 *>(lds);
    __syncthreads();
#pragma unroll
    for (int u = 0; u < NSUB; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const f32x16 &c = acc[u / kTN][u % kTN];
        red[(((wm * kWGK + wk) * NSUB + u) * 4 + e) * 64 + lane] = f32x4{c[4 * e], c[4 * e + 1], c[4 * e + 2], c[4 * e + 3]};
      }
    __syncthreads();
    f32x4 v[NSUB];
    bool bad = missed != 0;
#pragma unroll
    for (int g = 0; g < NSUB; ++g) {
      v[g] = red[((wm * kWGK) * NSUB * 4 + wk * NSUB + g) * 64 + lane];
#pragma unroll
      for (int k = 1; k < kWGK; ++k) v[g] += red[((wm * kWGK + k) * NSUB * 4 + wk * NSUB + g) * 64 + lane];
#pragma unroll
      for (int e = 0; e < 4; ++e) bad |= !__builtin_isfinite(v[g][e]);
    }
    // group g of this wave: rows 8*ge + 4*lg .. +3 of sub-tile u, column lr
    const int g0 = wk * NSUB;
    if (__syncthreads_or(bad)) {
      // a result that is not finite, or an operand the parts do not hold, somewhere in the tile: again in fp32, from memory
      // straight to the matrix instruction (lane l: row l%32, four of eight channels), 32 channels of a tap at a time and the
      // next 32 in flight.  Where two waves share a sub-tile, they take every other 32.
      constexpr int kShare = 4 / NSUB;
      const int u = g0 / 4, i = u / kTN, j = u % kTN;
      const int m = m0 + wm * WTM + i * 32 + lr, oc = n0 + j * 32 + lr;
      int vm = valid[0];
      if constexpr (TM == 2) vm = i ? valid[1] : valid[0];
      f32x4 x[2][4], y[2][4];
      int t = 0, c0 = 0;       // tap and first channel requested next
      auto request_fp32 = [&](int set) {
        const int d = ((t / 3 - 1) * W + t % 3 - 1) * (MODE == kBwd ? -1 : 1);
        const bool x_ok = t < 9 && ((vm >> t) & 1), y_ok = t < 9 && oc < a.OC;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int ch = c0 + k * 8 + lg * 4;   // IC is a multiple of four
          unsigned xo = x_ok && ch < IC ? (unsigned)((m + d) * IC + ch) * 4u : kOOB;
          unsigned yo = y_ok && ch < IC ? (unsigned)((oc * 9 + t) * IC + ch) * 4u : kOOB;
          asm("" : "+v"(xo), "+v"(yo));
          x[set][k] = buffer_load_16B(rin, xo);
          y[set][k] = buffer_load_16B(rwt, yo);
        }
#pragma unroll
        for (int k = 0; k < kShare; ++k) {
          c0 += 32;
          if (c0 >= IC) { c0 = 0; ++t; }
        }
      };
      f32x16 c;
#pragma unroll
      for (int e = 0; e < 16; ++e) c[e] = 0.f;
      if (kShare == 2 && (wk & 1)) {
        c0 = 32;
        if (c0 >= IC) { c0 = 0; ++t; }
      }
      const int batches = 9 * ((IC + 31) / 32);
      request_fp32(0);
      for (int it = 0; it < batches; it += 2 * kShare) {   // behind the last one: zeros
#pragma unroll
        for (int set = 0; set < 2; ++set) {
          request_fp32(set ^ 1);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int k = 0; k < 4; ++k) Elem<float>::mma(c, x[set][k], y[set][k]);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      if constexpr (NSUB == 4) {
#pragma unroll
        for (int g = 0; g < 4; ++g) v[g] = f32x4{c[4 * g], c[4 * g + 1], c[4 * g + 2], c[4 * g + 3]};
      } else {   // to each of the two its rows of the other's sums, through LDS behind the output tile
        static_assert(kTile + 8 * 2 * 64 * 16 <= kBytes, "exchanged sums fit");
        f32x4 *const half = reinterpret_cast<f32x4 *>(lds + kTile);
        const bool odd = wk & 1;
#pragma unroll
        for (int g = 0; g < 2; ++g) {
          f32x4 other;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float first = c[4 * g + e], second = c[8 + 4 * g + e];
            v[g][e] = odd ? second : first;
            other[e] = odd ? first : second;
          }
          half[(wave * 2 + g) * 64 + lane] = other;
        }
        __syncthreads();
#pragma unroll
        for (int g = 0; g < 2; ++g) v[g] += half[((wave ^ 1) * 2 + g) * 64 + lane];
      }
    }
#pragma unroll
    for (int g = 0; g < NSUB; ++g) {
      const int u = (g0 + g) / 4, ge = (g0 + g) % 4;
      const int row = wm * WTM + (u / kTN) * 32 + ge * 8 + lg * 4, col = (u % kTN) * 32 + lr;
#pragma unroll
      for (int e = 0; e < 4; ++e) Cs[row + e][col] = v[g][e];
    }
  });
}

template <int BM, int MODE>
int launch(EvalArgs a, hipStream_t st, StatParts *tiles_m_out) {
  a.tiles_m = (a.Mrows + BM - 1) / BM;
  a.tiles_n = (a.OC + kBN - 1) / kBN;
  if (tiles_m_out) { tiles_m_out->parts = a.tiles_m; tiles_m_out->rows = BM; }
  a.div_plane = make_fastdiv((unsigned)(a.IH * a.IW)); a.div_w = make_fastdiv((unsigned)a.IW);
  a.div_tn = make_fastdiv((unsigned)a.tiles_n);
  const long long grid = (long long)a.tiles_m * a.tiles_n;
  if (grid <= 0 || grid > 0x7fffffffLL) return set_error(RESIST_ESHAPE, "conv3 grid %lld", grid);
  {
    static const std::string label = std::string("conv3_f32_") + (MODE == kFwd ? "fwd_" : MODE == kEval ? "eval_" : "bwd_") + std::to_string(BM) + "x64";
    const double flops = 2.0 * a.Mrows * a.OC * a.IC * 9;
    const double bytes = 4.0 * ((double)a.Mrows * a.IC + (double)a.Mrows * a.OC * (1 + (a.addend ? 1 : 0) + (a.relu_mask ? 1 : 0) + (MODE == kBwd && a.bn_sums ? 1 : 0) +
                                (MODE == kEval ? (a.out ? 1 : 0) + (a.act_res ? 1 : 0) : 0)) + (double)a.OC * 9 * a.IC);
    prof::Scope ps(label.c_str(), flops, bytes, st);
    hipLaunchKernelGGL((conv3_split_kernel<BM, MODE>), dim3((unsigned)grid), dim3(kNT), 0, st, static_cast<const ArgsOf<MODE> &>(a));
  }
  RESIST_CHECK_LAUNCH("conv3");
  return RESIST_OK;
}

// 64-pixel tiles where 128-pixel ones would not give every CU a workgroup (512 ch 4x4, batch 128: 128 tiles)
template <int MODE>
int pick(const EvalArgs &a, hipStream_t st, StatParts *p) {
  const long long t128 = (long long)((a.Mrows + 127) / 128) * ((a.OC + kBN - 1) / kBN);
  return t128 >= 256 ? launch<128, MODE>(a, st, p) : launch<64, MODE>(a, st, p);
}

}  // namespace

// From 48 input channels: a chunk is 64 of them, however many there are.  us, fp32 instruction and here, 32x32, batch 128: 32 ->
// 32 channels 49 and 62, 48 -> 48 87 and 65.  (40 and 44 channels, which no network of this library can have, 87 and 62.)  And
// images no wider than the staged range allows.
bool conv3_takes(const IgemmArgs &a) {
  return a.R == 3 && a.S == 3 && a.stride == 1 && a.pad == 1 && a.IW <= kMaxW && a.IC >= 48;
}

int conv3_launch(const EvalArgs &a, int mode, hipStream_t st, StatParts *tiles_m_out) {
  return mode == kFwd ? pick<kFwd>(a, st, tiles_m_out) : mode == kBwd ? pick<kBwd>(a, st, tiles_m_out) : pick<kEval>(a, st, tiles_m_out);
}

}  // namespace resist
