// Weight gradient of a 3x3 stride-1 convolution of fp32 tensors on the bf16 matrix core (three bf16 parts per operand,
// six products, small terms first; results that are not finite, and operands too small for the parts, through a second
// pass on the fp32 instruction: see conv3.hip; all tiles twice, batch 128: 161 to 188 us, with one load in flight 202 to 358).
//
//   dW[k][r][s][c] = sum over pixels m of dY[m][k] * X[m + (r-1)*W + (s-1)][c]     (X of a tap off the image is zero)
//
// A workgroup owns 64 x 64 channels of all nine taps and a range of pixels: every pixel of dY and X is taken apart and
// staged once for nine taps (one tap at a time, as a plain split-K GEMM does it, staging costs more than the products).
// X rows live in a ring of 256 pixels, of which the 32 of a chunk and the W + 1 before and behind them are in use.
// Twelve waves: wave (r, kq, cq) accumulates the three taps of filter row r for one 32 x 32 quadrant of the channels.
// Both operands arrive pixel by pixel with the channels contiguous and are read back through the LDS transpose read.
//
// Measured with the reduction of the partial sums, us, fp32 instruction a tap at a time -> this kernel:
//   batch 128: 64 ch 32x32  96 -> 56    128 ch 16x16  96 -> 55    256 ch 8x8  101 -> 56    512 ch 4x4  111 -> 56
//   batch  77: 64 ch 32x32  62 -> 41    128 ch 16x16  63 -> 41    256 ch 8x8   65 -> 43    512 ch 4x4   78 -> 44
// The products are 32 us of it at the 1.75 GHz that the shader holds under them (23 at the nominal clock); the 38 MB of partial
// sums of 256 workgroups, written and read back, about 15.  Error against float64: 2e-8 to 1.3e-7, before 2e-8 to 4.9e-7.
#include "conv_tile.h"

namespace resist {
namespace {

constexpr int kNT = 768, kCh = 32, kRing = 256;
constexpr int kMirror = 6;                 // ring rows repeated behind its end: a tap's rows are at fixed offsets from the first
constexpr int kPart = 128;                 // bytes of one part (64 channels) of a staged row
constexpr int kPitch = 3 * kPart + 64;     // four consecutive rows fall on disjoint banks of a transpose read
constexpr int kStage = kCh * kPitch;

struct Wgrad3Args {
  const float *dy, *x;
  float *out;               // [splits][K][9][C]
  int M, W, H, C, K, rows_per_split, tiles_c, tiles;
  FastDiv div_tiles, div_tc, div_plane, div_w;
};

__global__ __launch_bounds__(kNT) void wgrad3_split_kernel(Wgrad3Args a) {
  // dY stages, X ring and the first rows of it again, zero rows, tap validity of the staged pixels
  __shared__ __attribute__((aligned(16))) char lds[2 * kStage + (kRing + 2 * kMirror + 1) * kPitch];
  __shared__ unsigned short taps_ok[2][kCh];
  char *const Xs = lds + 2 * kStage;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int fr = wave >> 2, kq = (wave >> 1) & 1, cq = wave & 1;   // filter row, channel quadrant
  // tiles fastest: the workgroups that share a range of pixels share an L2
  const int bid = xcd_contiguous(blockIdx.x, gridDim.x);
  const int split = fdiv(bid, a.div_tiles), tile = bid - split * a.tiles;
  const int tk = fdiv(tile, a.div_tc), tc = tile - tk * a.tiles_c;
  const int k0 = tk * 64, c0 = tc * 64, W = a.W;
  const int mbeg = split * a.rows_per_split, mend = min(a.M, mbeg + a.rows_per_split);
  const int chunks = (mend - mbeg + kCh - 1) / kCh;

  const __amdgpu_buffer_rsrc_t rdy = make_rsrc(a.dy, (unsigned)mend * a.K * 4u);   // rows of other splits: zeros
  const __amdgpu_buffer_rsrc_t rx = make_rsrc(a.x, (unsigned)a.M * a.C * 4u);

  // ---- staging: threads 0..511, 16 lanes (4 channels each) per row, one row of dY and one of X per chunk
  const bool stager = wave < 8;
  const int srow = (tid >> 4) & 31, sch = (tid & 15) * 4;
  // byte offsets of this thread's piece of dY row mbeg and of ring row 0 (pixel mbeg - W - 1).  A channel past the last one
  // starts at kOOB; pixels before the first and past the last of the tensor come back as zeros too (offsets wrap above its
  // size).  Where a tensor is so large that such an offset comes round to it, the value read belongs to a channel or a tap
  // that is not used.
  const unsigned dyo = k0 + sch < a.K ? (unsigned)((mbeg + srow) * a.K + k0 + sch) * 4u : kOOB;
  const unsigned xo = c0 + sch < a.C ? (unsigned)((mbeg - W - 1 + srow) * a.C + c0 + sch) * 4u : kOOB;
  f32x4 rd = {0.f, 0.f, 0.f, 0.f}, rxv = {0.f, 0.f, 0.f, 0.f};
  unsigned long long missed = 0;   // operands that three parts do not hold
  int xrow = 0, dyrow = 0;   // ring row and dY row (from mbeg) requested next
  auto request_x = [&]() { rxv = buffer_load_16B(rx, xo + (unsigned)(xrow * a.C) * 4u); };
  auto request = [&]() {
    rd = buffer_load_16B(rdy, dyo + (unsigned)(dyrow * a.K) * 4u);
    request_x();
    dyrow += kCh;
    xrow += kCh;
  };
  auto store_dy = [&](int stage) {
    char *d = lds + stage * kStage + srow * kPitch + sch * 2;
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      if (p == 2) split_check(rd, missed);
      *reinterpret_cast<u32x2 *>(d + p * kPart) = split_part(rd);
    }
  };
  auto store_x = [&](int row) {
    const int slot = (row + srow) & (kRing - 1);
    char *d = Xs + slot * kPitch + sch * 2;
    u32x2 v[3];
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      if (p == 2) split_check(rxv, missed);
      *reinterpret_cast<u32x2 *>(d + p * kPart) = v[p] = split_part(rxv);
    }
    if (slot < kMirror) {
#pragma unroll
      for (int p = 0; p < 3; ++p) *reinterpret_cast<u32x2 *>(d + kRing * kPitch + p * kPart) = v[p];
    }
  };
  // which taps of pixel m read inside its image
  auto taps_of = [&](int m) {
    const int n = fdiv(m, a.div_plane), rem = m - n * (a.H * W);
    const int h = fdiv(rem, a.div_w), w = rem - h * W;
    const int rows = (h > 0 ? 1 : 0) | 2 | (h + 1 < a.H ? 4 : 0), cols = (w > 0 ? 1 : 0) | 2 | (w + 1 < W ? 4 : 0);
    int v = 0;
#pragma unroll
    for (int r = 0; r < 3; ++r) v |= (rows >> r) & 1 ? cols << (3 * r) : 0;
    return v;
  };

  // ---- fragments.  Lane l supplies row 8*(l/32) + (l%16)/4 (and that + 4) of a 16-pixel k-step and columns
  // 16*((l/16)%2) + 4*(l%4) .. +3 of a 32-channel tile, and receives column l%32 of rows 8*(l/32) .. +7
  const int frow = (lane >> 5) * 8 + ((lane & 15) >> 2);
  const int fcol = (((lane >> 4) & 1) * 16 + (lane & 3) * 4) * 2;
  const int acol = frow * kPitch + kq * 64 + fcol, bcol = cq * 64 + fcol;
  constexpr int kZero = (kRing + kMirror) * kPitch;
  bf16x8 fa0[2], fa[3], fb[2][3];   // the filter-row tiles of a part in slots 0 and 1 in turn
  int baddr[3][2];
  auto fetch_a = [&](int set, int q, int at) {
    const char *p = lds + at + acol + q * kPart;
    const bf16x8 v = lds_read_tr_pair(p, p + 4 * kPitch);
    if (q == 0) fa0[set] = v;
    else fa[q] = v;
  };
  auto fetch_b = [&](int slot, int q) {
#pragma unroll
    for (int s = 0; s < 3; ++s)
      fb[slot][s] = lds_read_tr_pair(Xs + baddr[s][0] + s * kPitch + q * kPart, Xs + baddr[s][1] + (s + 4) * kPitch + q * kPart);
  };
  int ok0 = 0, ok1 = 0;    // validity bits of filter row fr for this lane's two rows of the k-step aimed at next
  auto fetch_ok = [&](int stage, int ks) {
    ok0 = taps_ok[stage][ks * 16 + frow] >> (3 * fr);
    ok1 = taps_ok[stage][ks * 16 + frow + 4] >> (3 * fr);
  };
  auto aim = [&](int row) {   // row: ring row of this lane's first pixel at tap (fr, 0)
    const int at = (row & (kRing - 1)) * kPitch;
#pragma unroll
    for (int s = 0; s < 3; ++s) {
      const int v0 = (ok0 << (31 - s)) >> 31, v1 = (ok1 << (31 - s)) >> 31;
      baddr[s][0] = ((at & v0) | (kZero & ~v0)) + bcol;
      baddr[s][1] = ((at & v1) | (kZero & ~v1)) + bcol;
    }
  };

  // Two accumulators a tap: the five products with a small factor add up apart from the leading one, so that a sum is
  // rounded at its full size once per 16 pixels
  f32x16 acc[3], small[3];
#pragma unroll
  for (int s = 0; s < 3; ++s)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[s][e] = small[s][e] = 0.f;
  auto product = [&](f32x16 (&sum)[3], bf16x8 pa, int slot) {
#pragma unroll
    for (int s = 0; s < 3; ++s) sum[s] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(pa, fb[slot][s], sum[s], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto lds_barrier = [&]() {
    __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
  };
  auto taps_to_lds = [&](int stage, int m) {
    if (tid < kCh) taps_ok[stage][tid] = (unsigned short)(m + tid < mend ? taps_of(m + tid) : 0);   // (no infinity past the end times 0)
  };

  // the ring up to the last row chunk 0 needs: rows 0 .. 2W + 33
  for (int i = tid; i < (kMirror + 1) * kPitch / 4; i += kNT) *reinterpret_cast<unsigned *>(Xs + (kRing + kMirror) * kPitch + i * 4) = 0;
  const int ahead = (2 * W + 2 + kCh - 1) / kCh * kCh;   // whole passes of X rows staged before chunk 0's own
  if (stager) {
    for (; xrow < ahead; xrow += kCh) {
      request_x();
      store_x(xrow);
    }
    request();             // dY of chunk 0, X rows ahead .. ahead + 31
    store_dy(0);
    store_x(ahead);
    request();
  }
  taps_to_lds(0, mbeg);
  lds_barrier();
  fetch_ok(0, 0);
  aim(frow + fr * W);
#pragma unroll
  for (int q = 0; q < 3; ++q) fetch_a(0, q, 0);
  fetch_b(0, 2);
  fetch_ok(0, 1);
  __builtin_amdgcn_sched_barrier(0);

  // Two k-steps of six product groups per chunk.  A part is fetched once its registers have served their last product:
  // the parts of X one after the other into two slots, those of dY for the next k-step.  The next chunk goes to LDS
  // during the first k-step; the barrier stands before the first fetch that reaches into it.
  for (int it = 0; it < chunks; ++it) {
    const int st = (it & 1) * kStage, nst = kStage - st;
    const int row = it * kCh + frow + fr * W;
    // ---- k-step 0: part 2 of X is in slot 0
    fetch_b(1, 1);
    product(small, fa0[0], 0);
    fetch_b(0, 0);
    if (stager) store_dy(nst ? 1 : 0);
    product(small, fa0[0], 1);
    product(small, fa[1], 1);
    aim(row + 16);
    fetch_b(1, 2);
    if (stager) store_x(ahead + (it + 1) * kCh);
    product(small, fa[2], 0);
    fetch_a(1, 2, st + 16 * kPitch);
    fetch_a(1, 0, st + 16 * kPitch);
    taps_to_lds((it + 1) & 1, mbeg + (it + 1) * kCh);
    product(small, fa[1], 0);
    fetch_a(1, 1, st + 16 * kPitch);
    product(acc, fa0[0], 0);
    // ---- k-step 1: part 2 of X is in slot 1 (behind the last chunk, the fetches for the next bring rows nobody uses)
    fetch_b(0, 1);
    if (stager) request();
    product(small, fa0[1], 1);
    fetch_b(1, 0);
    product(small, fa0[1], 0);
    lds_barrier();
    fetch_ok((it + 1) & 1, 0);
    product(small, fa[1], 0);
    aim(row + kCh);
    fetch_b(0, 2);
    fetch_ok((it + 1) & 1, 1);
    product(small, fa[2], 1);
    fetch_a(0, 2, nst);
    fetch_a(0, 0, nst);
    product(small, fa[1], 1);
    fetch_a(0, 1, nst);
    product(acc, fa0[1], 1);
  }

#pragma unroll
  for (int s = 0; s < 3; ++s) acc[s] += small[s];
  bool bad = missed != 0;
#pragma unroll
  for (int s = 0; s < 3; ++s)
#pragma unroll
    for (int e = 0; e < 16; ++e) bad |= !__builtin_isfinite(acc[s][e]);
  const int lr = lane & 31, lg = lane >> 5;
  const int c = c0 + cq * 32 + lr;
  if (__syncthreads_or(bad)) {
    // a result that is not finite, or an operand the parts do not hold, somewhere in the tile: again in fp32, from memory
    // straight to the matrix instruction, eight pixels at a time and the next eight in flight
    const int k = k0 + kq * 32 + lr;
    float d[2][4], x[2][4][3];
    int m2 = mbeg;           // pixel requested next
    auto request_fp32 = [&](int set) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int m = m2 + 2 * i + lg;
        const int n = fdiv(m, a.div_plane), rem = m - n * (a.H * W);
        const int h = fdiv(rem, a.div_w), w = rem - h * W;
        const bool in = m < mend && (unsigned)(h + fr - 1) < (unsigned)a.H;
        unsigned o = m < mend && k < a.K ? (unsigned)(m * a.K + k) * 4u : kOOB;
        asm("" : "+v"(o));
        d[set][i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rdy, (int)o, 0, 0));
#pragma unroll
        for (int s = 0; s < 3; ++s) {
          o = in && (unsigned)(w + s - 1) < (unsigned)W && c < a.C ? (unsigned)((m + (fr - 1) * W + s - 1) * a.C + c) * 4u : kOOB;
          asm("" : "+v"(o));
          x[set][i][s] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rx, (int)o, 0, 0));
        }
      }
      m2 += 8;
    };
#pragma unroll
    for (int s = 0; s < 3; ++s)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[s][e] = 0.f;
    request_fp32(0);
    while (m2 - 8 < mend) {   // behind an odd number of eights: zeros
#pragma unroll
      for (int set = 0; set < 2; ++set) {
        request_fp32(set ^ 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int s = 0; s < 3; ++s) acc[s] = __builtin_amdgcn_mfma_f32_32x32x2f32(d[set][i], x[set][i][s], acc[s], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  float *out = a.out + (size_t)split * a.K * 9 * a.C;
#pragma unroll
  for (int s = 0; s < 3; ++s)
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int k = k0 + kq * 32 + (e >> 2) * 8 + lg * 4 + (e & 3);
      if (k < a.K && c < a.C) out[((size_t)k * 9 + fr * 3 + s) * a.C + c] = acc[s][e];
    }
}

// ---- bf16 tensors: one filter row per workgroup -----------------------------------------------------------------------
//
// With one part an operand costs no arithmetic to stage, and the partial sums of nine taps per workgroup would take longer
// than the products; with one tap per workgroup (wgrad_bf16_kernel) every pixel comes from the L2 nine times.  Here a
// workgroup owns 64 x 64 channels of the three taps of one filter row: tap s of pixel m is pixel m + (r-1)*W + s - 1, so the
// 64 pixels of a chunk and one on either side serve three taps.  X rows live in a ring as above.  Eight waves: four
// quadrants of the channels, two halves of a chunk's pixels, added through LDS at the end.
//
// Measured with the reduction of the partial sums, us, one tap -> one filter row per workgroup, alone:
//   batch 128: 256 ch 8x8 29.1 -> 28.7    128 ch 16x16 28.7 -> 29.3    64 ch 32x32 27.9 -> 27.5    512 ch 4x4 32.9 -> 25.6
//   batch 64:  256 ch 14x14 38.7 -> 33.7  128 ch 28x28 36.3 -> 32.5    64 ch 56x56 36.6 -> 32.8
// It is bound by the LDS reads of the fragments, 1.3 per product.  Beside the data gradients of a step, which are short of L2
// bandwidth, it gains more: CIFAR-shaped model, batch 128, 5.89 -> 5.65 ms.
constexpr int kRowNT = 512, kRowCh = 64, kRowRing = 256, kRowPitch = kPart + 64;

struct WgradRowArgs {
  const void *dy, *x;
  float *out;               // [splits][K][9][C]
  int M, W, H, C, K, rows_per_split, tiles_c, tiles;
  FastDiv div_tiles, div_tc, div_plane, div_w;
};

__global__ __launch_bounds__(kRowNT) void wgrad3_row_bf16_kernel(WgradRowArgs a) {
  constexpr int kDyStage = kRowCh * kRowPitch;
  __shared__ __attribute__((aligned(16))) char lds[2 * kDyStage + (kRowRing + 2 * kMirror + 1) * kRowPitch];
  __shared__ unsigned char taps_ok[2][kRowCh];
  static_assert(2 * kDyStage + kRowRing * kRowPitch >= 4 * 3 * 4096, "half of the accumulators fits");
  char *const Xs = lds + 2 * kDyStage;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int half = wave >> 2, kq = (wave >> 1) & 1, cq = wave & 1;
  // tiles fastest, then filter rows: the workgroups that share a range of pixels share an L2
  const int bid = xcd_contiguous(blockIdx.x, gridDim.x);
  const int sr = fdiv(bid, a.div_tiles), tile = bid - sr * a.tiles;
  const int split = sr / 3, fr = sr - split * 3;
  const int tk = fdiv(tile, a.div_tc), tc = tile - tk * a.tiles_c;
  const int k0 = tk * 64, c0 = tc * 64, W = a.W;
  const int mbeg = split * a.rows_per_split, mend = min(a.M, mbeg + a.rows_per_split);
  const int chunks = (mend - mbeg + kRowCh - 1) / kRowCh;

  const __amdgpu_buffer_rsrc_t rdy = make_rsrc(a.dy, (unsigned)a.M * a.K * 2u);
  const __amdgpu_buffer_rsrc_t rx = make_rsrc(a.x, (unsigned)a.M * a.C * 2u);

  // ---- staging: 8 lanes (8 channels each) per row, one row of dY and one of X per thread and chunk
  const int srow = tid >> 3, sch = (tid & 7) * 8;
  const bool k_ok = k0 + sch < a.K, c_ok = c0 + sch < a.C;
  const int xpix = mbeg + (fr - 1) * W - 1 + srow;   // pixel of ring row srow
  f32x4 rd[2], rxv[2];
  int xrow = 0, dyrow = 0;
  auto load = [&](__amdgpu_buffer_rsrc_t r, unsigned o) {
    asm("" : "+v"(o));   // a selected offset; left alone, the compiler makes two loads behind a branch
    return buffer_load_16B(r, o);
  };
  auto request_x = [&](int set) {
    const int m = xpix + xrow;
    rxv[set] = load(rx, c_ok && (unsigned)m < (unsigned)a.M ? (unsigned)(m * a.C + c0 + sch) * 2u : kOOB);
    xrow += kRowCh;
  };
  auto request_dy = [&](int set) {
    const int m = mbeg + dyrow + srow;
    rd[set] = load(rdy, k_ok && m < mend ? (unsigned)(m * a.K + k0 + sch) * 2u : kOOB);
    dyrow += kRowCh;
  };
  auto store_dy = [&](int stage, int set) { *reinterpret_cast<f32x4 *>(lds + stage * kDyStage + srow * kRowPitch + sch * 2) = rd[set]; };
  auto store_x = [&](int row, int set) {
    const int slot = (row + srow) & (kRowRing - 1);
    char *d = Xs + slot * kRowPitch + sch * 2;
    *reinterpret_cast<f32x4 *>(d) = rxv[set];
    if (slot < kMirror) *reinterpret_cast<f32x4 *>(d + kRowRing * kRowPitch) = rxv[set];
  };
  // which taps of this filter row read inside the image of pixel m
  auto taps_to_lds = [&](int stage, int m0) {
    if (tid < kRowCh) {
      const int m = m0 + tid;
      const int n = fdiv(m, a.div_plane), rem = m - n * (a.H * W);
      const int h = fdiv(rem, a.div_w), w = rem - h * W;
      const bool in = m < mend && (unsigned)(h + fr - 1) < (unsigned)a.H;
      taps_ok[stage][tid] = (unsigned char)(in ? (w > 0 ? 1 : 0) | 2 | (w + 1 < W ? 4 : 0) : 0);
    }
  };

  // ---- fragments, as above; this wave's pixels of a chunk start at half * 32
  const int frow = (lane >> 5) * 8 + ((lane & 15) >> 2);
  const int fcol = (((lane >> 4) & 1) * 16 + (lane & 3) * 4) * 2;
  const int acol = (half * 32 + frow) * kRowPitch + kq * 64 + fcol, bcol = cq * 64 + fcol;
  constexpr int kZero = (kRowRing + kMirror) * kRowPitch;
  bf16x8 fa[2], fb[2][3];
  int ok[2][2];   // per k-step: tap bits of this lane's two pixels
  auto fetch_ok = [&](int stage) {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      ok[ks][0] = taps_ok[stage][half * 32 + ks * 16 + frow];
      ok[ks][1] = taps_ok[stage][half * 32 + ks * 16 + frow + 4];
    }
  };
  auto fetch = [&](int ks, int stage, int it) {
    const char *p = lds + stage * kDyStage + acol + ks * 16 * kRowPitch;
    fa[ks] = lds_read_tr_pair(p, p + 4 * kRowPitch);
    const int at = ((it * kRowCh + half * 32 + ks * 16 + frow) & (kRowRing - 1)) * kRowPitch;
#pragma unroll
    for (int s = 0; s < 3; ++s) {
      const int b0 = ((ok[ks][0] >> s) & 1 ? at : kZero) + bcol, b1 = ((ok[ks][1] >> s) & 1 ? at : kZero) + bcol;
      fb[ks][s] = lds_read_tr_pair(Xs + b0 + s * kRowPitch, Xs + b1 + (s + 4) * kRowPitch);
    }
  };
  f32x16 acc[3];
#pragma unroll
  for (int s = 0; s < 3; ++s)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[s][e] = 0.f;
  auto product = [&](int ks) {
#pragma unroll
    for (int s = 0; s < 3; ++s) acc[s] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[ks], fb[ks][s], acc[s], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto lds_barrier = [&]() {
    __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
  };

  // Chunk t needs ring rows 64 t .. 64 t + 65, i.e. passes t and t + 1 of X.  Behind chunk t wait, in register set (t + 1) % 2,
  // dY of chunk t + 1 and pass t + 2; those of chunk t + 2 are in flight.
  request_x(0); request_x(1); request_dy(0);
  for (int i = tid; i < (kMirror + 1) * kRowPitch / 4; i += kRowNT) *reinterpret_cast<unsigned *>(Xs + kZero + i * 4) = 0;
  taps_to_lds(0, mbeg);
  store_x(0, 0); store_x(kRowCh, 1); store_dy(0, 0);
  request_dy(1); request_x(1);
  request_dy(0); request_x(0);
  lds_barrier();
  fetch_ok(0);
  fetch(0, 0, 0);
  __builtin_amdgcn_sched_barrier(0);
  auto chunk = [&](int set, int it) {
    const int st = it & 1;
    fetch(1, st, it);
    store_dy(st ^ 1, set);
    store_x((it + 2) * kRowCh, set);
    taps_to_lds(st ^ 1, mbeg + (it + 1) * kRowCh);
    request_dy(set);
    request_x(set);
    __builtin_amdgcn_sched_barrier(0);
    product(0);
    lds_barrier();
    fetch_ok(st ^ 1);
    fetch(0, st ^ 1, it + 1);   // behind the last chunk: zeros nobody uses
    __builtin_amdgcn_sched_barrier(0);
    product(1);
  };
  for (int it = 0; it < chunks; it += 2) {   // behind an odd number of them: one without a valid pixel
    chunk(1, it);
    chunk(0, it + 1);
  }

  // the second half's sums go to the first
  __syncthreads();
  f32x4 *const red = reinterpret_cast<f32x4 *>(lds);
  if (half == 1) {
#pragma unroll
    for (int s = 0; s < 3; ++s)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        red[(((wave & 3) * 3 + s) * 4 + g) * 64 + lane] = f32x4{acc[s][4 * g], acc[s][4 * g + 1], acc[s][4 * g + 2], acc[s][4 * g + 3]};
  }
  __syncthreads();
  if (half == 1) return;
  const int lr = lane & 31, lg = lane >> 5, c = c0 + cq * 32 + lr;
  float *out = a.out + (size_t)split * a.K * 9 * a.C;
#pragma unroll
  for (int s = 0; s < 3; ++s)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const f32x4 o = red[((wave * 3 + s) * 4 + g) * 64 + lane];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int k = k0 + kq * 32 + g * 8 + lg * 4 + e;
        if (k < a.K && c < a.C) out[((size_t)k * 9 + fr * 3 + s) * a.C + c] = acc[s][4 * g + e] + o[e];
      }
    }
}

}  // namespace

constexpr int kWgrad3MaxW = 56;

// From 2^14 pixels, counted once for every 64 x 64 channels: below that the one-tap kernel's nine times as many workgroups
// win, most where the reduction of a layer is short.  us, one tap -> here: 64 ch 56x56, batch 1 12.6 -> 16.8, batch 4 21.5 -> 25.8,
// 32x32, batch 14 21.4 -> 25.9, batch 16 (the first taken) 27.0 -> 27.3; 128 ch 4x4, batch 80 14.3 -> 19.2, 8x8, batch 64 (taken)
// 26.4 -> 25.6; 256 ch 14x14, batch 1 9.3 -> 16.6; 16 ch 16x16, batch 64 (taken) 21.7 -> 17.9.  And from 640 pixels, unless the
// one-tap kernel would take 128 x 128 channels: with 64 x 64 it needs no split of that few, 304 -> 496 ch 4x4, batch 26 23.4 ->
// 25.1, 432 ch 16x16, batch 2 27.7 -> 32.2, but 448 ch 32x32, batch 1 45.3 -> 39.1, 512 ch 4x4, batch 16 28.2 -> 22.1.
bool wgrad3_takes(const ConvGeom &g) {
  const long long M = (long long)g.N * g.H * g.W, tiles = (long long)((g.K + 63) / 64) * ((g.C + 63) / 64);
  return g.R == 3 && g.S == 3 && g.stride == 1 && g.pad == 1 && g.W <= kWgrad3MaxW && M * tiles >= 1 << 14 &&
         (M >= 640 || wgrad_tile(g) == 128);
}

int wgrad3_launch(const ConvGeom &g, const float *dy, const float *x, float *out, int splits, int rows_per_split, hipStream_t st) {
  Wgrad3Args a{};
  a.dy = dy; a.x = x; a.out = out;
  a.M = g.N * g.H * g.W; a.W = g.W; a.H = g.H; a.C = g.C; a.K = g.K; a.rows_per_split = rows_per_split;
  a.tiles_c = (g.C + 63) / 64;
  a.tiles = a.tiles_c * ((g.K + 63) / 64);
  a.div_tiles = make_fastdiv((unsigned)a.tiles); a.div_tc = make_fastdiv((unsigned)a.tiles_c);
  a.div_plane = make_fastdiv((unsigned)(g.H * g.W)); a.div_w = make_fastdiv((unsigned)g.W);
  if (rows_per_split < kCh || rows_per_split % kCh || (long long)splits * rows_per_split < a.M ||
      (long long)(splits - 1) * rows_per_split >= a.M)
    return set_error(RESIST_EINVAL, "wgrad3: %d splits of %d rows for %d rows", splits, rows_per_split, a.M);
  hipLaunchKernelGGL(wgrad3_split_kernel, dim3((unsigned)(a.tiles * splits)), dim3(kNT), 0, st, a);
  RESIST_CHECK_LAUNCH("wgrad3");
  return RESIST_OK;
}

// From 2^28 products a tap, or where the tiles of the three rows nearly fill the chip by themselves: one split, no partial
// sums (512 -> 512 channels, batch 8 at 7x7: 22.5 -> 11.8 us, batch 16 at 4x4: 10.7 -> 9.1).  Below that the one-tap
// kernel's nine times as many workgroups win: 256 ch 8x8, batch 16 15.2 there, 16.0 here; 128 ch 28x28, batch 8 17.2 and 20.
// Not between 192 and 512 workgroups of a reduction beyond 2^30 padded products: one split of them leaves compute units idle
// for its whole length, and with more the partial sums take what they save (512 -> 512 channels at 14x14, us, one tap | one
// split | four: batch 32 55 | 64 | 55, batch 64 89 | 121 | 92; at 7x7, batch 64, the largest taken, 39.5 | 38.7 | 39.9).
bool wgrad3_row_takes(const ConvGeom &g) {
  const long long M = (long long)g.N * g.H * g.W, tiles = (long long)((g.K + 63) / 64) * ((g.C + 63) / 64);
  if (tiles >= 64 && tiles < 171 && M * tiles > 1 << 18) return false;
  return g.R == 3 && g.S == 3 && g.stride == 1 && g.pad == 1 && (M * g.K * g.C >= 1LL << 28 || (long long)g.K * g.C >= 1LL << 18);
}

int wgrad3_row_launch(const ConvGeom &g, const void *dy, const void *x, float *out, int splits, int rows_per_split, hipStream_t st) {
  WgradRowArgs a{};
  a.dy = dy; a.x = x; a.out = out;
  a.M = g.N * g.H * g.W; a.W = g.W; a.H = g.H; a.C = g.C; a.K = g.K; a.rows_per_split = rows_per_split;
  a.tiles_c = (g.C + 63) / 64;
  a.tiles = a.tiles_c * ((g.K + 63) / 64);
  a.div_tiles = make_fastdiv((unsigned)a.tiles); a.div_tc = make_fastdiv((unsigned)a.tiles_c);
  a.div_plane = make_fastdiv((unsigned)(g.H * g.W)); a.div_w = make_fastdiv((unsigned)g.W);
  const long long grid = (long long)a.tiles * 3 * splits;
  if (rows_per_split < 1 || (long long)splits * rows_per_split < a.M || (long long)(splits - 1) * rows_per_split >= a.M || grid > 0x7fffffffLL)
    return set_error(RESIST_EINVAL, "wgrad3 rows: %d splits of %d rows for %d rows", splits, rows_per_split, a.M);
  hipLaunchKernelGGL(wgrad3_row_bf16_kernel, dim3((unsigned)grid), dim3(kRowNT), 0, st, a);
  RESIST_CHECK_LAUNCH("wgrad3_row");
  return RESIST_OK;
}

}  // namespace resist
