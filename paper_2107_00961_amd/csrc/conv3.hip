// 3x3 stride-1 convolution, forward and data gradient, on a filter laid out beforehand for the matrix instruction: fp32 tensors on
// the bf16 matrix core, and bf16 tensors.
//
// Every fp32 operand a is taken apart into three bf16 numbers, a = h + m + l, each the nearest bf16 to what the ones
// before it leave: 8 + 8 + 8 significant bits, so nothing of a's 24 is lost.  A product is then six bf16 products
//   a*b = h*h' + (h*m' + m*h') + (m*m' + h*l' + l*h')      (what is left out is at most 2^-24 of |a*b|, 2^-27.5 in the mean)
// accumulated in fp32, small terms first.  v_mfma_f32_32x32x16_bf16 does 16 times the work of
// v_mfma_f32_32x32x2_f32 per cycle, so six of them take 6/16 of the time one fp32 product takes.
//
// Where that is not so, a workgroup computes its tile again on the fp32 matrix instruction: where a result is not finite
// (an infinity, or a finite value that rounds to one, leaves a NaN in the difference a - h and so in every output it
// reaches, and h*h' may overflow where a*b, within 0.8 % of the largest float, does not), and where it has an
// operand of so small a magnitude (below 2^-110; from 2^-103 up never) that its parts run out of bf16's bits: pixels are looked at
// as they are staged, of a filter prepare_filters leaves one word per 64x64 channels and tap.
//
// Pixels are staged once per 64 channels and serve all nine taps: the tile is a range of BM consecutive pixels of the flattened
// [N*H*W], tap (r, s) of pixel m is pixel m + (r-1)*W + (s-1), so a range of BM + 2W + 2 pixels holds every tap, whatever H, W
// and the image boundaries are; a tap that falls off its image reads a row of zeros instead.  The filter is not staged at all: a
// wave's tile is all pixels by 32 channels, so that a fragment of the filter is used by one wave, which loads it from
// where prepare_filters left it, 1 KB in lane order, three taps ahead.  Without filter rows to take apart and to
// pass through LDS per tap there is no barrier but the one per 64 channels, and the LDS holds two sets of pixels: the next one is
// staged between the products.
//
// What bounds it now, 256 channels 8x8, batch 128, fp32, 46 us (57 with the filter through LDS, 82 on the fp32 instruction): the
// products, 36 us of it at the clock that the shader holds under them (without any operand fetched in the loop it takes 43), and 8 us
// of a launch without products (first pixels, exchange of the four slices, epilogue).  bf16, the same layer: 14.5 us (18.7 with both
// operands through LDS), 5.8 of them without products.
//
// Measured, us, filter through LDS (bf16: igemm_kernel) -> this kernel, forward | data gradient:
//   fp32 batch 128: 64 ch 32x32  74 -> 64 | 74 -> 67    128 ch 16x16  64 -> 53 | 66 -> 56
//                  256 ch  8x8   60 -> 47 | 58 -> 48    512 ch  4x4   67 -> 47 | 67 -> 48
//   fp32 batch  77: 64 ch 32x32  54 -> 48 | 56 -> 48    128 ch 16x16  55 -> 37 | 55 -> 38
//                  256 ch  8x8   63 -> 33 | 63 -> 33    512 ch  4x4   59 -> 39 | 58 -> 39
//   bf16           256 ch 8x8, batch 128  18.7 -> 14.5 | 19.4 -> 14.5    512 ch 4x4, batch 128  22 -> 14.4 | 24.4 -> 14.1
//                  256 ch 14x14, batch 64 26.1 -> 24.3 | 28.6 -> 24.6    512 ch 7x7, batch 64   31.8 -> 21.6 | 34.2 -> 21.9
// Error against float64 over 27 to 4608 products per output: 1.3e-7 to 4.6e-7 (2-norm), the fp32 instruction's 2.5e-7 to
// 1.1e-6.
#include <algorithm>

#include "conv_tile.h"

namespace resist {
namespace {

constexpr int kWidest = 56;
constexpr int kBN = 64, kNT = 512, kBK = 64, kWK = 4;
constexpr int kRing = 3;      // taps of filter fragments in registers
constexpr int kAhead = 4;     // filter pieces of 8 KB a workgroup asks for up front

// 8 waves: 2 along the output channels, 4 sharing the reduction (wave slice k takes 16 of every 64 channels).  A wave's tile is
// all BM pixels by 32 channels, so a filter fragment is used by one wave only and comes straight from memory.
// ROWS (fp32): on the filter as it is stored, or for a data gradient its transpose, rows [output channel][tap][IC], which a wave takes
// apart as it goes: the same products in the same order, for calls with no room for the fragments.  us, with the filter through LDS -> this,
// forward | data gradient with the transposition: batch 128, 64 ch 32x32 65.5 -> 63.0 | 68.6 -> 68.4, 128 ch 16x16 55.5 -> 52.5 |
// 59.3 -> 57.9, 256 ch 8x8 51.1 -> 48.2 | 56.3 -> 54.7, 512 ch 4x4 61.2 -> 51.9 | 68.5 -> 57.4, batch 64, 64 ch 56x56 109.8 -> 105.8 |
// 113.1 -> 113.0, 128 ch 28x28 105.4 -> 95.4 | 108.8 -> 101.1.
template <int NP, int BM, int NBUF, int kMaxW, int MODE, bool ROWS>
__global__ __launch_bounds__(kNT, NP == 3 ? 2 : 4) void conv3_kernel(Conv3Args<MODE> a) {
  using T = std::conditional_t<NP == 3, float, __bf16>;
  constexpr int ES = sizeof(T), VEC = 16 / ES;
  constexpr int TM = BM / 32;
  constexpr int kPlane = kBK * 2, kPitch = NP * kPlane + 16;
  constexpr int LPR = kBK / VEC;                        // lanes per staged row
  constexpr int RPP = kNT / LPR;                        // rows per staging pass
  constexpr int PX = BM + 2 * kMaxW + 2;
  constexpr int PA = (PX + RPP - 1) / RPP;
  constexpr int LDC = kBN + 8;
  constexpr int kBuf = PX * kPitch;
  constexpr size_t kOperand = (size_t)NBUF * kBuf + kPitch;   // staged pixels; the row behind them is zero
  constexpr size_t kRound1 = (size_t)8 * 2 * TM * 1024, kRound2 = kRound1 / 2;
  constexpr size_t kTile = sizeof(float) * BM * LDC;
  constexpr size_t kEnd = kRound2 + kTile > kRound1 ? kRound2 + kTile : kRound1;
  constexpr size_t kBytes = kOperand > kEnd ? kOperand : kEnd;
  __shared__ __attribute__((aligned(16))) char lds[kBytes];
  __shared__ int row_off[BM];
  char *const Px = lds;
  float (*Cs)[LDC] = reinterpret_cast<float (*)[LDC]>(lds + kRound2);

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wk = wave & 3, wn = wave >> 2;
  const int lr = lane & 31, lg = lane >> 5;
  const int bid = xcd_contiguous(blockIdx.x, gridDim.x);
  int tm, tn;
  if (a.m_fast) { tn = fdiv(bid, a.div_tm); tm = bid - tn * a.tiles_m; }
  else { tm = fdiv(bid, a.div_tn); tn = bid - tm * a.tiles_n; }
  const int m0 = tm * BM, n0 = tn * kBN;
  const int W = a.IW, IC = a.IC, px = BM + 2 * W + 2;   // staged pixels: m0 - W - 1 .. m0 + BM + W
  const int cchunks = a.cchunks;

  for (int r = tid; r < BM; r += kNT) row_off[r] = m0 + r < a.Mrows ? m0 + r : -1;

  // ---- staging
  const __amdgpu_buffer_rsrc_t rin = make_rsrc(a.in, (unsigned)a.N * a.IH * W * IC * ES);
  const int srow = tid / LPR, sch = (tid % LPR) * VEC;
  char *const pdst = Px + srow * kPitch + sch * 2;
  // pixels before the first and past the last of the tensor come back as zeros (offsets wrap above the size)
  const unsigned poff = (unsigned)((m0 - W - 1 + srow) * IC + sch) * ES;
  f32x4 rp[PA];
  unsigned long long missed = 0;   // operands that three parts do not hold
  auto request_pixels = [&](int pc) {
    const bool ok = pc * kBK + sch < IC;
#pragma unroll
    for (int i = 0; i < PA; ++i) {
      unsigned o = ok && i * RPP + srow < px ? poff + (unsigned)(i * RPP * IC + pc * kBK) * ES : kOOB;
      asm("" : "+v"(o));   // a selected offset; left alone, the compiler makes two loads behind a branch and waits for each
      rp[i] = buffer_load_16B(rin, o);
    }
  };
  auto store_pixels = [&](int i, int buf) {
    if ((i + 1) * RPP <= PX || i * RPP + srow < PX) {
      char *row = pdst + buf + i * RPP * kPitch;
      if constexpr (NP == 3) {
        f32x4 v = rp[i];
#pragma unroll
        for (int p = 0; p < 3; ++p) {
          if (p == 2) split_check(v, missed);
          *reinterpret_cast<u32x2 *>(row + p * kPlane) = split_part(v);
        }
      } else {
        *reinterpret_cast<f32x4 *>(row) = rp[i];
      }
    }
  };
  request_pixels(0);
  unsigned flagged = 0;            // filter rows of this tile that three parts do not hold
  if constexpr (NP == 3 && !ROWS)
    for (int i = tid; i < a.cchunks * 9; i += kNT) flagged |= a.flags[tn * a.cchunks * 9 + i];

  // ---- filter fragments: [octile of 32][chunk][tap][wave slice][part][64 lanes][16 bytes]
  const int chunk_bytes = 9 * kWK * NP * 1024;
  const char *wbase = static_cast<const char *>(a.frag) + (size_t)(tn * 2 + wn) * a.cchunks * chunk_bytes;
  const __amdgpu_buffer_rsrc_t rwt = ROWS ? make_rsrc(a.wt, (unsigned)a.OC * 9u * IC * 4u) : make_rsrc(wbase, (unsigned)(a.cchunks * chunk_bytes));
  const int woff = wk * NP * 1024 + lane * 16;
  // rows: lane l reads output channel l % 32, channels 8 * (l / 32) .. +7 of the wave's slice.  The values wait in `raw` and become
  // the parts of the next tap during the products of this one.
  static_assert(!ROWS || NP == 3, "filters in fp32");
  const int wch = wk * 16 + lg * 8, woc = n0 + wn * 32 + lr;
  const unsigned wrow = woc < a.OC ? (unsigned)(woc * 9 * IC + wch) * 4u : kOOB;
  f32x4 fb[ROWS ? 2 : kRing][NP], raw[ROWS ? kRing : 1][2];
  auto fetch_b = [&](int slot, int t, int c) {   // tap t of chunk c, both uniform
    if constexpr (ROWS) {
      const int left = IC - c * kBK - wch;   // a multiple of four
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        unsigned o = left > h * 4 ? wrow + (unsigned)(c * kBK + h * 4) * 4u : kOOB;
        asm("" : "+v"(o));
        raw[slot][h] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rwt, (int)o, t * IC * 4, 0));
      }
    } else {
#pragma unroll
      for (int p = 0; p < NP; ++p)
        fb[slot][p] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rwt, woff + p * 1024, c * chunk_bytes + t * kWK * NP * 1024, 0));
    }
  };
  unsigned long long wmissed = 0;
  auto take_part = [&](int set, int slot, int p) {   // in order
    if constexpr (ROWS) {
      if (p == 2) {
        split_check(raw[slot][0], wmissed);
        split_check(raw[slot][1], wmissed);
        asm("" : "+s"(wmissed));   // left alone, the compiler keeps every mask to the end, in lanes of vector registers
      }
      const u32x2 x = split_part(raw[slot][0]), y = split_part(raw[slot][1]);
      fb[set][p] = __builtin_bit_cast(f32x4, u32x4{x[0], x[1], y[0], y[1]});
    }
  };
#pragma unroll
  for (int t = 0; t < kRing; ++t) fetch_b(t, t, 0);
  // Three taps of bf16 products are over before a line arrives from beyond the L2, and all workgroups of an XCD walk the filter
  // in step.  So those that share it ask for a part each, up front.  us a layer of a step, without -> with: 256 ch 8x8 and 512 ch
  // 4x4 (the mean of a network's 50), batch 64 16.5 -> 14.8, batch 128 20.7 -> 20.2, 512 ch 7x7 with 256 ch 14x14, batch 16
  // 19.3 -> 17.9, batch 64 29.4 -> 28.5.
  f32x4 ahead[NP == 1 ? kAhead : 1];
  if constexpr (NP == 1) {
    const int first = (tm % a.share) * a.ahead * kNT * 16 + tid * 16;
    const __amdgpu_buffer_rsrc_t rall = make_rsrc(static_cast<const char *>(a.frag) + (size_t)tn * 2 * a.cchunks * chunk_bytes, (unsigned)(2 * a.cchunks * chunk_bytes));
#pragma unroll
    for (int i = 0; i < kAhead; ++i) ahead[i] = buffer_load_16B(rall, i < a.ahead ? (unsigned)(first + i * kNT * 16) : kOOB);
  }

  // which taps of this lane's pixels lie inside their image, and where in LDS its operands start
  int valid[TM], abase[TM];
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int ml = i * 32 + lr, m = m0 + ml;
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
  const int zbase = NBUF * kBuf + wk * 32 + lg * 16;
  if (tid < kPitch / 4) *reinterpret_cast<unsigned *>(Px + NBUF * kBuf + tid * 4) = 0;

  f32x16 acc[TM];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[i][e] = 0.f;

  auto lds_barrier = [&]() {
    __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
  };

#pragma unroll
  for (int i = 0; i < PA; ++i) store_pixels(i, 0);
  if constexpr (ROWS) {
#pragma unroll
    for (int p = 0; p < 3; ++p) take_part(0, 0, p);
    fetch_b(0, kRing, 0);
  }
  lds_barrier();

  // ---- one chunk of 64 channels, nine taps.  The pixel fragments of a tap are fetched during the products of the tap before it,
  // each part as soon as its last product is issued; only the leading parts, which the last product of a tap and the second of the
  // next both use, have two register sets.  MORE: the next chunk's pixels are staged beside the products.
  f32x4 fa0[2][TM], fa[NP][TM];
  int at[TM];
  auto aim = [&](int t, int here) {
    const int d = ((t / 3 - 1) * W + t % 3 - 1) * (MODE == kBwd ? -kPitch : kPitch) + here;
#pragma unroll
    for (int i = 0; i < TM; ++i) at[i] = (valid[i] >> t) & 1 ? abase[i] + d : zbase;
  };
  auto fetch_a = [&](int set, int q) {
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const f32x4 v = *reinterpret_cast<const f32x4 *>(Px + at[i] + q * kPlane);
      if (q == 0) fa0[set][i] = v;
      else fa[q][i] = v;
    }
  };
  auto product = [&](int set, int slot, int pa, int pb) {
#pragma unroll
    for (int i = 0; i < TM; ++i) Elem<__bf16>::mma(acc[i], pa == 0 ? fa0[set][i] : fa[pa][i], fb[slot][pb]);
#pragma unroll
    for (int i = 0; i < TM; ++i) {   // what else is to be done here goes between the products
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  auto chunk = [&](auto more_tag, int c) {
    constexpr bool MORE = decltype(more_tag)::value;
    // (left alone, the compiler keeps the addresses of all nine taps in registers)
#pragma unroll
    for (int i = 0; i < TM; ++i) asm("" : "+v"(valid[i]), "+v"(abase[i]));
    const int here = NBUF == 2 && (c & 1) ? kBuf : 0, there = NBUF == 2 ? kBuf - here : 0;
    aim(0, here);
    if constexpr (NP == 3) fetch_a(0, 2);
    fetch_a(0, 0);
    if constexpr (NP == 3) fetch_a(0, 1);
    if (MORE) request_pixels(c + 1);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < 9; ++t) {
      const int set = t & 1, nx = set ^ 1, slot = ROWS ? set : t % kRing, later = (t + 1) % kRing;
      auto next_part = [&](int p) {
        if (t < 8 || MORE) take_part(nx, later, p);
      };
      auto stage = [&](int third) {   // passes are spread over taps 2 to 8
        if constexpr (MORE && NBUF == 2) {
#pragma unroll
          for (int i = 0; i < PA; ++i)
            if (t >= 2 && i * 7 / PA == t - 2 && i % 3 == third) store_pixels(i, there);
        }
      };
      if (t < 8) aim(t + 1, here);
      if constexpr (NP == 3) {
        stage(0);
        product(set, slot, 2, 0);
        if (t < 8) fetch_a(nx, 2);
        next_part(0);
        product(set, slot, 0, 2);
        if (t < 8) fetch_a(nx, 0);
        stage(1);
        product(set, slot, 1, 1);
        next_part(1);
        product(set, slot, 1, 0);
        if (t < 8) fetch_a(nx, 1);
        stage(2);
        product(set, slot, 0, 1);
        next_part(2);
        product(set, slot, 0, 0);
      } else {
        if (t < 8) fetch_a(nx, 0);
        stage(0); stage(1); stage(2);
        product(set, slot, 0, 0);
      }
      const int next = t + (ROWS ? kRing + 1 : kRing);
      if (next < 9 || MORE) fetch_b(ROWS ? later : slot, next % 9, c + next / 9);
    }
    if constexpr (ROWS && MORE) {
#pragma unroll
      for (int p = 0; p < 3; ++p) fb[0][p] = fb[1][p];
    }
    if (MORE) {
      lds_barrier();
      if constexpr (NBUF == 1) {
#pragma unroll
        for (int i = 0; i < PA; ++i) store_pixels(i, 0);
        lds_barrier();
      }
    }
  };
  for (int c = 0; c + 1 < cchunks; ++c) chunk(std::true_type{}, c);
  chunk(std::false_type{}, cchunks - 1);

  // A result that is not finite, or an operand the parts do not hold, somewhere in the tile: again on the fp32 instruction, from
  // memory straight to it (lane l: row l%32, four of eight channels), 32 channels of a tap at a time and the next 32 in flight.
  // Wave slice i computes the tile's pixels 32*i .. +31; of 64-pixel tiles two slices each, every other 32 channels.
  auto fp32_tile = [&]() {
    constexpr int kShare = TM <= 2 ? 2 : 1;
    static_assert(TM == 2 || TM == 3 || TM == 4, "slices of a tile");
    const int i = kShare == 2 ? wk & 1 : wk, share = kShare == 2 ? wk >> 1 : 0;
    const int m = m0 + i * 32 + lr, oc = n0 + wn * 32 + lr;
    const bool mine = i < TM;
    const __amdgpu_buffer_rsrc_t rw32 = make_rsrc(a.wt, (unsigned)a.OC * 9u * IC * 4u);
    int vm = 0;
#pragma unroll
    for (int k = 0; k < TM; ++k) vm = i == k ? valid[k] : vm;
    f32x4 x[2][4], y[2][4];
    int t = 0, c0 = 0;       // tap and first channel requested next
    auto next_channels = [&]() {
      c0 += 32;
      if (c0 >= IC) { c0 = 0; ++t; }
    };
    auto request_fp32 = [&](int set) {
      const int d = ((t / 3 - 1) * W + t % 3 - 1) * (MODE == kBwd ? -1 : 1);
      const bool x_ok = t < 9 && ((vm >> t) & 1), y_ok = t < 9 && oc < a.OC;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int ch = c0 + k * 8 + lg * 4;   // IC is a multiple of four
        unsigned xo = x_ok && ch < IC ? (unsigned)((m + d) * IC + ch) * 4u : kOOB;
        asm("" : "+v"(xo));
        x[set][k] = buffer_load_16B(rin, xo);
        if (MODE == kBwd && !ROWS) {   // the filter as it is stored, [IC][9][OC]
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            unsigned yo = y_ok && ch < IC ? (unsigned)(((ch + e) * 9 + t) * a.OC + oc) * 4u : kOOB;
            asm("" : "+v"(yo));
            y[set][k][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rw32, (int)yo, 0, 0));
          }
        } else {
          unsigned yo = y_ok && ch < IC ? (unsigned)((oc * 9 + t) * IC + ch) * 4u : kOOB;
          asm("" : "+v"(yo));
          y[set][k] = buffer_load_16B(rw32, yo);
        }
      }
#pragma unroll
      for (int k = 0; k < kShare; ++k) next_channels();
    };
    f32x16 c;
#pragma unroll
    for (int e = 0; e < 16; ++e) c[e] = 0.f;
    if (mine) {
      if (share) next_channels();
      const int batches = 9 * ((IC + 31) / 32);
      request_fp32(0);
      for (int it = 0; it < batches; it += 2 * kShare) {   // behind the last one: zeros
#pragma unroll
        for (int set = 0; set < 2; ++set) {
          request_fp32(set ^ 1);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int k = 0; k < 4; ++k) Elem<float>::mma(c, x[set][k], y[set][k] * a.wscale);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
    f32x4 *const other = reinterpret_cast<f32x4 *>(lds);   // the second share's sums, below the output tile
    if constexpr (kShare == 2) {
      static_assert((size_t)4 * 4 * 64 * 16 <= kRound2, "exchanged sums fit");
      if (share) {
#pragma unroll
        for (int g = 0; g < 4; ++g) other[((wn * 2 + i) * 4 + g) * 64 + lane] = f32x4{c[4 * g], c[4 * g + 1], c[4 * g + 2], c[4 * g + 3]};
      }
      __syncthreads();
    }
    if (mine && !share) {
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        f32x4 s = f32x4{c[4 * g], c[4 * g + 1], c[4 * g + 2], c[4 * g + 3]};
        if constexpr (kShare == 2) s += other[((wn * 2 + i) * 4 + g) * 64 + lane];
#pragma unroll
        for (int e = 0; e < 4; ++e) Cs[i * 32 + g * 8 + lg * 4 + e][wn * 32 + lr] = s[e];
      }
    }
  };

  conv_epilogue<T, BM, kBN, kNT, MODE>(a, Cs, row_off, tm, n0, [&]() {
    // The four slices of a wave tile meet in two exchanges: with the neighbour slice, after which each holds half of the tile's
    // groups of four rows, then with the one two away.  Sums are (0 + 1) + (2 + 3).
    f32x4 *const red = reinterpret_cast<f32x4 *>(lds);
    const bool odd = wk & 1, high = wk & 2;
    auto group = [&](int g) {
      const f32x16 &c = acc[g >> 2];
      const int e = (g & 3) * 4;
      return f32x4{c[e], c[e + 1], c[e + 2], c[e + 3]};
    };
    auto either = [](bool second, const f32x4 &x, const f32x4 &y) {
      f32x4 r;
#pragma unroll
      for (int e = 0; e < 4; ++e) r[e] = second ? y[e] : x[e];
      return r;
    };
    if constexpr (NP == 1) {
#pragma unroll
      for (int i = 0; i < kAhead; ++i) asm volatile("" : : "v"(ahead[i]));
    }
    __syncthreads();
#pragma unroll
    for (int g = 0; g < 2 * TM; ++g) red[(wave * 2 * TM + g) * 64 + lane] = either(odd, group(g + 2 * TM), group(g));
    __syncthreads();
    f32x4 half[2 * TM], v[TM];
#pragma unroll
    for (int g = 0; g < 2 * TM; ++g) half[g] = either(odd, group(g), group(g + 2 * TM)) + red[((wave ^ 1) * 2 * TM + g) * 64 + lane];
    __syncthreads();
#pragma unroll
    for (int g = 0; g < TM; ++g) red[(wave * TM + g) * 64 + lane] = either(high, half[g + TM], half[g]);
    __syncthreads();
    bool bad = (missed | wmissed) != 0 || flagged != 0;
#pragma unroll
    for (int g = 0; g < TM; ++g) {
      v[g] = either(high, half[g], half[g + TM]) + red[((wave ^ 2) * TM + g) * 64 + lane];
      if constexpr (NP == 3) {
#pragma unroll
        for (int e = 0; e < 4; ++e) bad |= !__builtin_isfinite(v[g][e]);
      }
    }
    const int col = wn * 32 + lr;
    if constexpr (NP == 3) {
      if (__syncthreads_or(bad)) {
        fp32_tile();
        return;
      }
    }
    const int g0 = (odd ? 2 * TM : 0) + (high ? TM : 0);
#pragma unroll
    for (int g = 0; g < TM; ++g) {
      const int row = ((g0 + g) >> 2) * 32 + ((g0 + g) & 3) * 8 + lg * 4;
#pragma unroll
      for (int e = 0; e < 4; ++e) Cs[row + e][col] = v[g][e];
    }
  });
}

template <int NP, int BM, int NBUF, int MAXW, int MODE, bool ROWS>
int launch(Conv3Args<kEval> a, hipStream_t st, StatParts *tiles_m_out) {
  a.tiles_m = (a.Mrows + BM - 1) / BM;
  a.tiles_n = (a.OC + kBN - 1) / kBN;
  if (tiles_m_out) { tiles_m_out->parts = a.tiles_m; tiles_m_out->rows = BM; }
  a.div_plane = make_fastdiv((unsigned)(a.IH * a.IW)); a.div_w = make_fastdiv((unsigned)a.IW);
  a.div_tn = make_fastdiv((unsigned)a.tiles_n); a.div_tm = make_fastdiv((unsigned)a.tiles_m);
  const long long grid = (long long)a.tiles_m * a.tiles_n;
  if (grid <= 0 || grid > 0x7fffffffLL) return set_error(RESIST_ESHAPE, "conv3 grid %lld", grid);
  Conv3Args<MODE> k;
  static_cast<ArgsOf<MODE> &>(k) = a;
  k.frag = a.frag; k.flags = a.flags; k.wscale = a.wscale; k.cchunks = a.cchunks;
  k.m_fast = (long long)a.OC * 9 * a.IC * NP * 2 > (long long)a.Mrows * a.IC * (NP == 3 ? 4 : 2);
  const long long per_xcd = (grid + 7) / 8, sharing = k.m_fast ? std::min<long long>(per_xcd, a.tiles_m) : per_xcd / a.tiles_n;
  k.share = (int)std::max<long long>(1, sharing);
  k.ahead = (int)std::min<long long>(kAhead, (9LL * 8 * 1024 * NP * a.cchunks + (long long)k.share * kNT * 16 - 1) / ((long long)k.share * kNT * 16));
  {
    static const std::string label = std::string("conv3_") + (NP == 3 ? "f32_" : "bf16_") + (MODE == kFwd ? "fwd_" : MODE == kEval ? "eval_" : "bwd_") + std::to_string(BM) + "x64";
    const double flops = 2.0 * a.Mrows * a.OC * a.IC * 9;
    const double bytes = (NP == 3 ? 4.0 : 2.0) * ((double)a.Mrows * a.IC + (double)a.Mrows * a.OC * (1 + (a.addend ? 1 : 0) + (a.relu_mask ? 1 : 0) + (MODE == kBwd && a.bn_sums ? 1 : 0) +
                                (MODE == kEval ? (a.out ? 1 : 0) + (a.act_res ? 1 : 0) : 0)) + (double)a.OC * 9 * a.IC);
    prof::Scope ps(label.c_str(), flops, bytes, st);
    hipLaunchKernelGGL((conv3_kernel<NP, BM, NBUF, MAXW, MODE, ROWS>), dim3((unsigned)grid), dim3(kNT), 0, st, k);
  }
  RESIST_CHECK_LAUNCH("conv3");
  return RESIST_OK;
}

// fp32: one workgroup to a compute unit (LDS).  128-pixel tiles, or 64-pixel ones where those would not give every unit a
// tile.  In training steps, on whole chunks of channels and at least two of them, whichever of 128, 96 and 64 pixels leaves the units
// idle least, what a tile costs beside its products (8 of 46 us) being what 24 pixels cost: 256 ch 8x8, batch 77: 64 pixels 42, 96
// 33 us; 128 ch 16x16: 128 pixels 49, 96 37; batch 128: 96 pixels 65 and 61, 128 47 and 53.  (One
// chunk: 64 ch 32x32, batch 77 47.5 and 47.3, batch 100 57.9 and 55.3.  A last chunk that is not full, 96 ch 16x16 44.9 and 36.2, and
// the test-time forward, 128 ch 16x16, batch 77 47.5 and 37.4, would gain too; they stay in the tiles that they are tested in.)
// (Images wider than 32: the pixels of 128 are staged once at a time.  us, kernel with the filter through LDS -> this one, data gradient with
// its filter's preparation: batch 64, 64 ch 56x56 113.2 -> 106.2, batch 16, 128 ch 56x56 110.3 -> 101.6, 48x48 82.8 -> 76.2, 40x40
// 54.7 -> 51.2; 96 pixels at 40x40 60.4, 64 pixels 57.3.)  bf16: 64-pixel tiles, two workgroups to a unit; 128-pixel
// ones with one, 256 ch 8x8, batch 128: 16.5 us.
template <int MODE, bool ROWS>
int pick(const Conv3Args<kEval> &a, int dt, hipStream_t st, StatParts *p) {
  if constexpr (!ROWS) {
    if (dt == DT_BF16) return launch<1, 64, 2, 56, MODE, false>(a, st, p);
  }
  auto tiles = [&](int bm) { return (long long)((a.Mrows + bm - 1) / bm) * ((a.OC + kBN - 1) / kBN); };
  int bm = tiles(128) >= 256 ? 128 : 64;
  if (a.IW > 32) return bm == 128 ? launch<3, 128, 1, 56, MODE, ROWS>(a, st, p) : launch<3, 64, 2, 56, MODE, ROWS>(a, st, p);
  if constexpr (MODE != kEval) {
    if (a.IC >= 2 * kBK && a.IC % kBK == 0) {
      auto cost = [&](int bm) { return (tiles(bm) + 255) / 256 * (bm + 24); };
      bm = cost(128) <= cost(96) && cost(128) <= cost(64) ? 128 : cost(96) <= cost(64) ? 96 : 64;
      if (bm == 96) return launch<3, 96, 2, 32, MODE, ROWS>(a, st, p);
    }
  }
  return bm == 128 ? launch<3, 128, 2, 32, MODE, ROWS>(a, st, p) : launch<3, 64, 2, 32, MODE, ROWS>(a, st, p);
}

}  // namespace

// fp32 from 48 input channels: a chunk is 64 of them, however many there are (32 -> 32 channels, 32x32, batch 128: 49 us on the fp32
// instruction).  bf16 from 256: 128 ch 16x16 18 us here and 17 in igemm_kernel's tiles, 64 ch 32x32 24.5 and 22, and unless 128x128 tiles
// fill their two or more rounds of 256 workgroups well.  Time in those | here, by rounds of 512 tiles of 64x64 of which the last costs a
// third more than it holds; data gradients, us, with the filter's preparation, there | here: 256 -> 256 ch 16x16, batch 128 52.1 | 52.2, 32x32
// 180.7 | 190.0, 28x28, batch 64 88.6 | 79.7, 512 -> 256 ch 16x16, batch 128 95.9 | 99.1, 320 -> 320 87.7 | 76.3, 512 -> 512 14x14, batch 64
// 85.7 | 81.1.  Images no wider than the staged range allows, and filters whose 64 rows an offset reaches.
bool conv3_takes(const IgemmArgs &a, int dt) {
  if (dt == DT_BF16 && a.OC > 64) {
    const double k = 9.0 * a.IC;
    const long long t128 = (long long)((a.Mrows + 127) / 128) * ((a.OC + 127) / 128), t64 = (long long)((a.Mrows + 63) / 64) * ((a.OC + 63) / 64);
    const double rounds = (double)((t128 + 255) / 256), part = (double)(t64 % 512) / 512;
    const double here = 3 + ((double)(t64 / 512) + (part > 0 ? std::min(1.0, part + 0.3) : 0.0)) * (2.1 + 4.04e-3 * k);
    if (rounds >= 2 && 5 + rounds * (1.5 + 8.55e-3 * k) < here) return false;
  }
  return a.R == 3 && a.S == 3 && a.stride == 1 && a.pad == 1 && a.IW <= kWidest && a.IC >= (dt == DT_BF16 ? 256 : 48) && a.IC <= 8192;
}

int64_t conv3_filter_bytes(int OC, int IC, int dt) {
  const int64_t tiles = (int64_t)((OC + kBN - 1) / kBN) * ((IC + kBK - 1) / kBK) * 9;
  return tiles * 2 * kWK * 1024 * (dt == DT_BF16 ? 1 : 3) + (dt == DT_BF16 ? 0 : tiles * 4);
}

int conv3_launch(const EvalArgs &e, const Filter &w, int dt, int mode, hipStream_t st, StatParts *p) {
  Conv3Args<kEval> a;
  static_cast<EvalArgs &>(a) = e;
  a.cchunks = (e.IC + kBK - 1) / kBK;
  a.frag = w.prep;
  a.flags = reinterpret_cast<const unsigned *>(static_cast<const char *>(w.prep) + (int64_t)((e.OC + kBN - 1) / kBN) * a.cchunks * 9 * 2 * kWK * 3 * 1024);
  a.wscale = w.scale;
  return mode == kFwd ? pick<kFwd, false>(a, dt, st, p) : mode == kBwd ? pick<kBwd, false>(a, dt, st, p) : pick<kEval, false>(a, dt, st, p);
}

int conv3_launch_rows(const EvalArgs &e, int mode, hipStream_t st, StatParts *p) {
  Conv3Args<kEval> a;
  static_cast<EvalArgs &>(a) = e;
  a.cchunks = (e.IC + kBK - 1) / kBK;
  a.frag = nullptr;
  a.flags = nullptr;
  a.wscale = 1.f;
  return mode == kFwd ? pick<kFwd, true>(a, DT_F32, st, p) : pick<kBwd, true>(a, DT_F32, st, p);
}

}  // namespace resist
