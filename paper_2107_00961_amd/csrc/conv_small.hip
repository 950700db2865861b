// Convolutions whose output is too small to give every compute unit a large tile: small batches, late stages.
//
// Such a layer is bound by the length of the reduction that a workgroup walks alone (512 -> 512 channels at 7x7, one
// image: eight 64x64 tiles, 4608 products long, every 128 bytes of them a barrier and an exposed load).  Here a workgroup
// owns a 32x32 tile, so that there are four times as many, and its eight waves each take an eighth of the reduction,
// without a barrier between them until the eight partial tiles are added, in wave order, in LDS.
//
// A unit of work is 128 bytes of channels of one tap: 64 rows (32 pixels, 32 filter rows) of one cache line each, eight
// lanes to a line, two units in flight in registers, then through LDS of the wave's own to the matrix instruction's
// layout.  (Loaded straight into that layout a request touches 32 lines for 32 bytes each, and the kernel is bound by the
// lines the L1 looks up: 19.6 us for the layer above instead of 11.3, and no faster than the 64x64 tiles.)
//
// Measured, us, 64x64 tiles -> this kernel, forward, batch 1 and 8:
//   bf16 512 ch 7x7 20.8 -> 11.3, 21.1 -> 12.6    256 ch 8x8 12.3 -> 8.7, 12.7 -> 9.4    2048 -> 512 1x1 7x7 11.5 -> 7.8, 12.2 -> 8.7
//   fp32 512 ch 4x4 50.6 -> 26.0, 53.9 -> 27.1    256 ch 8x8 28.6 -> 16.8, 29.6 -> 18.0    16 ch 16x16 9.6 -> 6.9, 10.0 -> 7.1
// (fp32 on the fp32 instruction, which bounds the long ones: 17 of the 26 us.)  Error against float64: eight short sums
// instead of a long one, 0.9e-7 to 6.8e-7 where the 64x64 tiles have 1.8e-7 to 8.5e-7.
#include "conv_tile.h"

namespace resist {
namespace {

constexpr int kBM = 32, kBN = 32, kNW = 8, kNT = kNW * 64;
constexpr int kLDC = kBN + 8;
constexpr int kPitch = 128 + 16;   // consecutive rows 4 banks apart: conflict-free 16-byte reads

template <typename T, int MODE>
__global__ __launch_bounds__(kNT) void conv_small_kernel(ArgsOf<MODE> a) {
  using E = Elem<T>;
  constexpr int VEC = E::VEC, ES = (int)sizeof(T), BK = 8 * VEC;   // channels a unit
  constexpr int NS = 4;                                            // matrix steps a unit
  constexpr int kRows = kBM + kBN, kPasses = kRows / 8;            // staged rows of a wave, 8 lanes each
  __shared__ __attribute__((aligned(16))) char lds[kNW * kRows * kPitch];
  __shared__ int row_off[kBM];
  static_assert(kNW * kRows * kPitch >= kNW * 4096 + kBM * kLDC * 4, "partial tiles and the output tile fit");
  f32x4 (*const red)[4][64] = reinterpret_cast<f32x4 (*)[4][64]>(lds);                     // [kNW]
  float (*const Cs)[kLDC] = reinterpret_cast<float (*)[kLDC]>(lds + kNW * 4096);           // behind the partial tiles

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 31, lg = lane >> 5;
  const int bid = a.cls == 1 ? xcd_contiguous(blockIdx.x, gridDim.x) : (int)blockIdx.x;
  const int bq = fdiv(bid, a.div_tn);
  const int tn = bid - bq * a.tiles_n;
  const int cidx = fdiv(bq, a.div_tm);   // parity class of a stride-2 data gradient
  const int tm = bq - cidx * a.tiles_m;
  const int ph = a.cls == 2 ? cidx >> 1 : 0, pw = a.cls == 2 ? cidx & 1 : 0;
  const int m0 = tm * kBM, n0 = tn * kBN;

  // taps that contribute: r0, r0 + tstep, ... (all of them unless a stride-2 data gradient)
  int r0 = 0, s0 = 0, tstep = 1;
  if (MODE == kBwd && a.stride == 2) { r0 = (ph + a.pad) & 1; s0 = (pw + a.pad) & 1; tstep = 2; }
  const int nr = r0 < a.R ? (a.R - r0 + tstep - 1) / tstep : 0;
  const int ns = s0 < a.S ? (a.S - s0 + tstep - 1) / tstep : 0;
  const int cunits = (a.IC + BK - 1) / BK;
  const int units = nr * ns * cunits;
  const int begin = units * wave / kNW, end = units * (wave + 1) / kNW;   // this wave's share

  // rows this lane stages: centre pixel and where its channels start; the filter rows' starts
  const int srow = lane >> 3, sch = (lane & 7) * VEC;
  int hc[kBM / 8], wc[kBM / 8], aoff[kBM / 8], boff[kBN / 8];
#pragma unroll
  for (int i = 0; i < kBM / 8; ++i) {
    const int m = m0 + i * 8 + srow;
    const int n = fdiv(m, a.div_plane);
    const int rem = m - n * (a.OHc * a.OWc);
    const int ohc = fdiv(rem, a.div_w), owc = rem - ohc * a.OWc;
    if (MODE != kBwd) { hc[i] = ohc * a.stride - a.pad; wc[i] = owc * a.stride - a.pad; }
    else if (a.stride == 1) { hc[i] = ohc + a.pad; wc[i] = owc + a.pad; }
    else { hc[i] = ohc; wc[i] = owc; }
    aoff[i] = (((n * a.IH + hc[i]) * a.IW + wc[i]) * a.IC + sch) * ES;
    if (m >= a.Mrows) hc[i] = -(1 << 24);   // never in range
  }
#pragma unroll
  for (int i = 0; i < kBN / 8; ++i) {
    const int oc = n0 + i * 8 + srow;
    boff[i] = oc < a.OC ? (oc * a.R * a.S * a.IC + sch) * ES : (int)kOOB;   // stays past the end whatever tap is added
  }
  if (tid < kBM) {
    const int m = m0 + tid;
    const int n = fdiv(m, a.div_plane);
    const int rem = m - n * (a.OHc * a.OWc);
    const int ohc = fdiv(rem, a.div_w), owc = rem - ohc * a.OWc;
    row_off[tid] = m < a.Mrows ? (n * a.OH + ohc * a.cls + ph) * a.OW + owc * a.cls + pw : -1;
  }
  const __amdgpu_buffer_rsrc_t rin = make_rsrc(a.in, (unsigned)a.N * a.IH * a.IW * a.IC * ES);
  const __amdgpu_buffer_rsrc_t rwt = make_rsrc(a.wt, (unsigned)a.OC * a.R * a.S * a.IC * ES);

  // the unit requested next: tap, first channel
  int left = end - begin, c0, tr, ts;
  {
    const int tap = begin / cunits, tq = ns ? tap / ns : 0;
    c0 = (begin - tap * cunits) * BK;
    tr = r0 + tq * tstep;
    ts = s0 + (tap - tq * ns) * tstep;
  }
  f32x4 reg[2][kPasses];   // units in flight
  auto request = [&](int set) {
    int dh, dw;
    if (MODE != kBwd) { dh = tr; dw = ts; }
    else if (a.stride == 1) { dh = -tr; dw = -ts; }
    else { dh = (ph + a.pad - tr) >> 1; dw = (pw + a.pad - ts) >> 1; }   // even by construction
    const bool live = left > 0 && c0 + sch < a.IC;   // past the share: zeros
    const int da = ((dh * a.IW + dw) * a.IC + c0) * ES, db = ((tr * a.S + ts) * a.IC + c0) * ES;
#pragma unroll
    for (int i = 0; i < kBM / 8; ++i) {
      const bool ok = live && (unsigned)(hc[i] + dh) < (unsigned)a.IH && (unsigned)(wc[i] + dw) < (unsigned)a.IW;
      unsigned o = ok ? (unsigned)(aoff[i] + da) : kOOB;
      asm("" : "+v"(o));   // a selected offset; left alone, the compiler may make two loads behind a branch
      reg[set][i] = buffer_load_16B(rin, o);
    }
#pragma unroll
    for (int i = 0; i < kBN / 8; ++i) {
      unsigned o = live ? (unsigned)(boff[i] + db) : kOOB;
      asm("" : "+v"(o));
      reg[set][kBM / 8 + i] = buffer_load_16B(rwt, o);
    }
    --left;
    c0 += BK;
    const bool cwrap = c0 >= a.IC;
    c0 = cwrap ? 0 : c0;
    const bool swrap = cwrap && ts + tstep >= a.S;
    ts = cwrap ? (swrap ? s0 : ts + tstep) : ts;
    tr = swrap ? tr + tstep : tr;
  };
  // The staged rows belong to this wave alone and LDS accesses of a wave take place in their order: no barrier, and one
  // buffer: the next unit is written behind the reads of this one.  The lanes exchange them, so the order is one between
  // lanes and has to be told to the compiler (which emits nothing for it).
  auto wave_order = [&]() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  char *const mine = lds + wave * kRows * kPitch;
  char *const dst = mine + srow * kPitch + (lane & 7) * 16;
  const char *const src = mine + lr * kPitch + lg * 16;
  auto store = [&](int set) {
#pragma unroll
    for (int i = 0; i < kPasses; ++i) *reinterpret_cast<f32x4 *>(dst + i * 8 * kPitch) = reg[set][i];
  };

  f32x16 acc;
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[e] = 0.f;
  int cu = c0;   // first channel of the unit multiplied next
  auto unit = [&](int set) {
    f32x4 fa[NS], fb[NS];
    wave_order();
#pragma unroll
    for (int k = 0; k < NS; ++k) {
      fa[k] = *reinterpret_cast<const f32x4 *>(src + k * 32);
      fb[k] = *reinterpret_cast<const f32x4 *>(src + kBM * kPitch + k * 32);
    }
    wave_order();
    store(set);
    request(set);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < NS; ++k)
      if (cu + k * 2 * VEC < a.IC) E::mma(acc, fa[k], fb[k]);   // uniform: steps past the last channel are zeros
    cu = cu + BK >= a.IC ? 0 : cu + BK;
    __builtin_amdgcn_sched_barrier(0);
  };
  request(0);
  request(1);
  store(0);
  request(0);
  for (int it = begin; it < end; it += 2) {   // behind an odd share: a unit of zeros
    unit(1);
    unit(0);
  }

  __syncthreads();   // row_off; every wave is done with its staged rows
  conv_epilogue<T, kBM, kBN, kNT, MODE>(a, Cs, row_off, tm, n0, [&]() {
#pragma unroll
    for (int g = 0; g < 4; ++g) red[wave][g][lane] = f32x4{acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]};
    __syncthreads();
    if (wave < 4) {   // rows 8*wave + 4*lg .. +3, column lr
      f32x4 v = red[0][wave][lane];
#pragma unroll
      for (int w = 1; w < kNW; ++w) v += red[w][wave][lane];
#pragma unroll
      for (int e = 0; e < 4; ++e) Cs[wave * 8 + lg * 4 + e][lr] = v[e];
    }
  });
}

template <typename T, int MODE>
int launch(EvalArgs a, hipStream_t st, StatParts *tiles_m_out) {
  a.tiles_m = (a.Mrows + kBM - 1) / kBM;
  a.tiles_n = (a.OC + kBN - 1) / kBN;
  if (tiles_m_out) { tiles_m_out->parts = a.tiles_m; tiles_m_out->rows = kBM; }
  a.div_plane = make_fastdiv((unsigned)(a.OHc * a.OWc)); a.div_w = make_fastdiv((unsigned)a.OWc);
  a.div_tn = make_fastdiv((unsigned)a.tiles_n); a.div_tm = make_fastdiv((unsigned)a.tiles_m);
  const long long grid = (long long)a.tiles_m * a.tiles_n * a.cls * a.cls;
  if (grid <= 0 || grid > 0x7fffffffLL) return set_error(RESIST_ESHAPE, "conv_small grid %lld", grid);
  {
    static const std::string label = std::string("conv_small_") + (sizeof(T) == 4 ? "f32_" : "bf16_") + (MODE == kFwd ? "fwd" : MODE == kEval ? "eval" : "bwd");
    const double flops = 2.0 * a.N * (MODE != kBwd ? (double)a.OH * a.OW : (double)a.IH * a.IW) * a.OC * a.IC * a.R * a.S;
    const double bytes = sizeof(T) * ((double)a.N * a.IH * a.IW * a.IC + (double)a.N * a.OH * a.OW * a.OC * (1 + (a.addend ? 1 : 0) + (a.relu_mask ? 1 : 0) + (MODE == kBwd && a.bn_sums ? 1 : 0) +
                                       (MODE == kEval ? (a.out ? 1 : 0) + (a.act_res ? 1 : 0) : 0)) +
                                      (double)a.OC * a.R * a.S * a.IC);
    prof::Scope ps(label.c_str(), flops, bytes, st);
    hipLaunchKernelGGL((conv_small_kernel<T, MODE>), dim3((unsigned)grid), dim3(kNT), 0, st, static_cast<const ArgsOf<MODE> &>(a));
  }
  RESIST_CHECK_LAUNCH("conv_small");
  return RESIST_OK;
}

}  // namespace

// Up to one workgroup per compute unit (a 257th waits for a whole tile of another; 400 tiles: 1.0 times the 64x64 tiles'
// time at best, 800: twice it), and reductions long enough to be worth splitting: forward, one to 32 images, this kernel
// over the 64x64 tiles, in bf16 4608 products 11-13 over 20-21 us, 1152 7.5-8.2 over 8.4-8.7, 1024 6.6-7.0 over 8.0, but 576
// 7.0 over 6.8 and 256 6.3 over 5.4; in fp32 144 7.0 over 10.0, 256 8.2-8.6 over 9.6, 576 10.6-11.5 over 11.1-11.8, 4608 26-30
// over 51-56.
bool conv_small_takes(const IgemmArgs &a, int dt) {
  const int length = a.R * a.S * a.IC / (a.cls * a.cls);   // a parity class of a stride-2 data gradient: a quarter of the taps
  return conv_small_rows((long long)a.Mrows * a.cls * a.cls, a.OC, a.cls) && length >= (dt == DT_BF16 ? 1024 : 144);
}

bool conv_small_rows(long long pixels, int OC, int cls) {
  const long long m = pixels / (cls * cls);
  return (m + kBM - 1) / kBM * ((OC + kBN - 1) / kBN) * cls * cls <= 256;
}

int conv_small_launch(const EvalArgs &a, int dt, int mode, hipStream_t st, StatParts *p) {
  if (dt == DT_BF16)
    return mode == kFwd ? launch<__bf16, kFwd>(a, st, p) : mode == kBwd ? launch<__bf16, kBwd>(a, st, p) : launch<__bf16, kEval>(a, st, p);
  return mode == kFwd ? launch<float, kFwd>(a, st, p) : mode == kBwd ? launch<float, kBwd>(a, st, p) : launch<float, kEval>(a, st, p);
}

}  // namespace resist
