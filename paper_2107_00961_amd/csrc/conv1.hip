// Widening 1x1 convolutions of bf16 tensors, and the data gradients of narrowing ones: output channels at least twice the input
// channels, which are few.  They are bound by the output tensor (and, in a data gradient, by the addend, the mask and the BN input
// that are as large), and in 128x128 tiles by what every tile costs beside it: 12 us of a launch and 2.7 us per tile and compute unit.
//
// Here the filter stays and the pixels stream.  A wave owns 32 output channels, whose filter rows it keeps in registers, and a
// workgroup a range of pixels, 32 or 64 of them at a time through two LDS buffers that its waves share.  The filter is the
// left operand, so that a lane holds one pixel and, after the halves of the wave have traded fours of channels
// (v_permlane32_swap), 16-byte runs of channels: the output goes from the accumulators to memory, and the side inputs of the next 32
// pixels are requested before the products of these, so that no wait for them stands behind a store.  The per-channel sums
// of a BN (forward statistics, or the first pass of a backward) stay in registers for the whole range, in fp32 for 128 pixels at a
// time and from there in float64: one part per workgroup, for 56x56 and batch 64 349 forward and 242 backward where 128x128 tiles
// have 1568, for 28x28 157 and 392, for 14x14 79 and 98.  (In fp32 throughout, which loses bits with every doubling of the range:
// 64 -> 256 ch 56x56, batch 64, with its statistics 26.2 us, 27.4 this way; 128 -> 512 28x28 21.2 and 21.3.)
//
// Measured, us, 128x128 tiles -> this kernel:
//   forward        64 -> 256 ch 56x56, batch 64 44.7 -> 24.3 (5.3 TB/s)   128 -> 512 28x28 29.7 -> 19.5   256 -> 1024 14x14 22.0 -> 18.2
//   data gradient (no side inputs)                46.3 -> 31.9                          31.2 -> 22.8                       22.9 -> 20.5
//   forward        64 -> 256 ch 56x56, batch 8   9.9 -> 7.2    128 -> 512 28x28, batch 16 10.9 -> 9.2
#include <algorithm>

#include "conv_tile.h"

namespace resist {
namespace {

constexpr int kSumRows = 128;   // pixels whose BN sums are taken in fp32: no more than in a tile of the other kernels

// PX pixels a step; NW waves of 32 output channels each, KC * 16 input channels.  Registers allow three waves to a SIMD forward,
// two with the side inputs.
template <int KC, int NW, int PX, int MODE>
__global__ __launch_bounds__(NW * 64, MODE == kBwd ? 2 : 3) void conv1_stream_kernel(Conv1Args a) {
  constexpr int NT = NW * 64;
  constexpr int kPitch = KC * 32 + 16;                  // consecutive rows 4 banks apart
  constexpr int LPR = KC * 2, RPP = NT / LPR, PA = PX / RPP;   // staging: lanes per row, rows per pass, passes
  static_assert(NT % LPR == 0 && PX % RPP == 0 && PA >= 1 && PX % 32 == 0, "staging passes");
  __shared__ __attribute__((aligned(16))) char xs[2][PX * kPitch];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 31, lg = lane >> 5;
  const int bid = xcd_contiguous(blockIdx.x, gridDim.x);
  const int part = fdiv(bid, a.div_tn), tn = bid - part * a.tiles_n;
  const int IC = a.IC, OC = a.OC;
  const int m0 = part * a.rows, m1 = min(a.Mrows, m0 + a.rows);
  const int n0 = (tn * NW + wave) * 32;                 // this wave's channels

  const __amdgpu_buffer_rsrc_t rin = make_rsrc(a.in, (unsigned)m1 * IC * 2u);   // rows of other workgroups: zeros
  const __amdgpu_buffer_rsrc_t rwt = make_rsrc(a.wt, (unsigned)OC * IC * 2u);

  // ---- pixels
  const int srow = tid / LPR, spiece = tid % LPR;
  const bool sok = spiece * 8 < IC;
  f32x4 rp[PA];
  auto request = [&](int m) {
#pragma unroll
    for (int i = 0; i < PA; ++i) {
      unsigned o = sok ? (unsigned)((m + i * RPP + srow) * IC + spiece * 8) * 2u : kOOB;
      rp[i] = buffer_load_16B(rin, o);
    }
  };
  auto store = [&](int buf) {
#pragma unroll
    for (int i = 0; i < PA; ++i) *reinterpret_cast<f32x4 *>(&xs[buf][(i * RPP + srow) * kPitch + spiece * 16]) = rp[i];
  };
  request(m0);
  // ---- the filter stays in registers: lane l holds row l%32, channels 8*(l/32) .. +7 of every 16
  f32x4 w[KC];
#pragma unroll
  for (int k = 0; k < KC; ++k) {
    const int ch = k * 16 + lg * 8;
    unsigned o = n0 + lr < OC && ch < IC ? (unsigned)((n0 + lr) * IC + ch) * 2u : kOOB;
    asm("" : "+v"(o));
    w[k] = buffer_load_16B(rwt, o);
  }
  // A lane ends up with channels c0 .. c0+7 and c0+16 .. c0+23 of one pixel
  const int c0 = n0 + lg * 8;
  const bool ok0 = c0 < OC, ok1 = c0 + 16 < OC;         // OC is a multiple of 8
  const bool has_mask = MODE == kBwd && a.relu_mask != nullptr, has_bn = MODE == kBwd && a.bn_sums != nullptr;
  const bool sums = MODE == kFwd ? a.stats != nullptr : has_bn;
  // rows past the range and tensors that are not there: loads of zeros, stores of nothing
  const unsigned all = (unsigned)m1 * OC * 2u;
  const __amdgpu_buffer_rsrc_t rout = make_rsrc(a.out, all), radd = make_rsrc(a.addend, MODE == kBwd && a.addend ? all : 0u),
                               rmask = make_rsrc(a.relu_mask, has_mask ? all : 0u), rbn = make_rsrc(a.bn_y, has_bn ? all : 0u);
  const float pass = has_mask ? 0.f : -INFINITY;        // the mask's values have to be larger
  const unsigned ooff = ok0 ? (unsigned)((m0 + lr) * OC + c0) * 2u : kOOB, ooff1 = ok1 ? (unsigned)((m0 + lr) * OC + c0 + 16) * 2u : kOOB;
  constexpr int kSide = MODE == kBwd ? 2 : 1;
  f32x4 qa[kSide][2], qm[kSide][2], qy[kSide][2];       // of this and of the next 32 pixels
  auto request_side = [&](int set, unsigned d) {
    if constexpr (MODE == kBwd) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const unsigned o = (h ? ooff1 : ooff) + d;
        qa[set][h] = buffer_load_16B(radd, o);
        qm[set][h] = buffer_load_16B(rmask, o);
        qy[set][h] = buffer_load_16B(rbn, o);
      }
    }
  };
  float centre[16], s1[16], s2[16];
#pragma unroll
  for (int e = 0; e < 16; ++e) { centre[e] = 0.f; s1[e] = 0.f; s2[e] = 0.f; }
  if (has_bn) {
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int c = c0 + (e & 7) + (e >> 3) * 16;
      centre[e] = c < OC ? a.bn_mean[c] : 0.f;
    }
  }
  // Over the 32 pixels of a lane half: each step a lane hands half of its sums to a partner, whose number differs in the bit that is
  // looked at (and perhaps in lower ones), and takes the other half of the partner's: lane l ends with sum number l % 32 of its half.
  double total = 0;   // of the range so far
  auto add_up = [&]() {
    float v[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, s1[e]), __builtin_bit_cast(unsigned, s2[e]), false, false);
      const unsigned x = r[0], y = r[1];
      v[e] = __builtin_bit_cast(float, x) + __builtin_bit_cast(float, y);
      s1[e] = s2[e] = 0.f;
    }
    auto hand_over = [&](auto half_tag, auto partner_tag) {
      constexpr int half = decltype(half_tag)::value, partner = decltype(partner_tag)::value;
      const bool up = lane & half;
#pragma unroll
      for (int i = 0; i < half; ++i) {
        const float keep = up ? v[i + half] : v[i], give = up ? v[i] : v[i + half];
        v[i] = keep + __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, give), partner, 0xf, 0xf, true));
      }
    };
    hand_over(std::integral_constant<int, 8>{}, std::integral_constant<int, 0x140>{});   // row_mirror: lane ^ 15
    hand_over(std::integral_constant<int, 4>{}, std::integral_constant<int, 0x141>{});   // row_half_mirror: lane ^ 7
    hand_over(std::integral_constant<int, 2>{}, std::integral_constant<int, 0x1b>{});    // quad_perm 3 2 1 0
    hand_over(std::integral_constant<int, 1>{}, std::integral_constant<int, 0xb1>{});    // quad_perm 1 0 3 2
    total += (double)v[0];
  };
  request_side(0, 0);
  store(0);
  request(m0 + PX);
  __syncthreads();

  int buf = 0;
  for (int m = m0; m < m1; m += PX, buf ^= 1) {
#pragma unroll
    for (int t = 0; t < PX / 32; ++t) {
      const int sub = m - m0 + t * 32, cur = MODE == kBwd ? t & 1 : 0;
      const bool live = m0 + sub + lr < m1;
      const unsigned d = (unsigned)(sub * OC) * 2u;
      request_side(cur ^ 1, d + (unsigned)OC * 64u);   // (behind the range's last pixels: zeros)
      f32x16 acc;
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[e] = 0.f;
#pragma unroll
      for (int k = 0; k < KC; ++k) {
        const f32x4 x = *reinterpret_cast<const f32x4 *>(&xs[buf][(t * 32 + lr) * kPitch + k * 32 + lg * 16]);
        Elem<__bf16>::mma(acc, w[k], x);
      }
      // Lane l holds pixel l%32 and channels 8*(e/4) + 4*(l/32) + e%4.  The halves of the wave trade: the lower one gives its fours
      // of the odd groups of eight for the upper one's of the even groups.
#pragma unroll
      for (int g = 0; g < 4; g += 2)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float even = acc[4 * g + e], odd = acc[4 * g + 4 + e];
          const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, even), __builtin_bit_cast(unsigned, odd), false, false);
          const unsigned lo = r[0], hi = r[1];
          acc[4 * g + e] = __builtin_bit_cast(float, lo);
          acc[4 * g + 4 + e] = __builtin_bit_cast(float, hi);
        }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = acc[8 * h + e];
        if constexpr (MODE == kBwd) {
          float x[8];
          Vec<__bf16>::unpack(__builtin_bit_cast(u32x4, qa[cur][h]), x);
#pragma unroll
          for (int e = 0; e < 8; ++e) v[e] += x[e];
          Vec<__bf16>::unpack(__builtin_bit_cast(u32x4, qm[cur][h]), x);
#pragma unroll
          for (int e = 0; e < 8; ++e) v[e] = x[e] > pass ? v[e] : 0.f;
        }
        u32x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = pack_bf16x2(v[2 * e], v[2 * e + 1]);
        __builtin_amdgcn_raw_buffer_store_b128(o, rout, (int)((h ? ooff1 : ooff) + d), 0, 0);
        if (sums) {   // of the values as stored
          Vec<__bf16>::unpack(o, v);
          if (MODE == kFwd) {
            if (m == m0 && t == 0) {   // the range's first row
#pragma unroll
              for (int e = 0; e < 8; ++e) centre[8 * h + e] = __shfl(v[e], lane & 32, 64);
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              const float d = live ? v[e] - centre[8 * h + e] : 0.f;
              s1[8 * h + e] += d;
              s2[8 * h + e] = fmaf(d, d, s2[8 * h + e]);
            }
          } else {
            float y[8];
            Vec<__bf16>::unpack(__builtin_bit_cast(u32x4, qy[cur][h]), y);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              const float g = live ? v[e] : 0.f;
              s1[8 * h + e] += g;
              s2[8 * h + e] = fmaf(g, y[e] - centre[8 * h + e], s2[8 * h + e]);
            }
          }
        }
      }
    }
    store(buf ^ 1);
    request(m + 2 * PX);
    if (sums && ((m + PX - m0) % kSumRows == 0 || m + PX >= m1)) add_up();
    __syncthreads();
  }
  if (!sums) return;
  const int e = lr & 15, c = c0 + (e & 7) + (e >> 3) * 16, second = lr >> 4;
  if (c < OC) {
    if (MODE == kFwd) {
      a.stats[((size_t)(1 + second) * a.parts + part) * OC + c] = (float)total;
    } else {
      a.bn_sums[((size_t)second * a.parts + part) * OC + c] = (float)(second ? total * (double)a.bn_invstd[c] : total);
    }
  }
  if (MODE == kFwd) {   // the shifts, from whichever lane: the first of each half writes its sixteen
    if (lr == 0)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int ch = c0 + (i & 7) + (i >> 3) * 16;
        if (ch < OC) a.stats[(size_t)part * OC + ch] = centre[i];
      }
  }
}

template <int KC, int NW, int PX, int MODE>
int launch(const IgemmArgs &g, hipStream_t st, StatParts *p) {
  Conv1Args a;
  static_cast<IgemmArgs &>(a) = g;
  a.tiles_n = (g.OC + NW * 32 - 1) / (NW * 32);
  a.div_tn = make_fastdiv((unsigned)a.tiles_n);
  // a range of pixels per workgroup, as many workgroups as are resident at once
  const long long want = std::max(1, 256 * 4 * (MODE == kBwd ? 2 : 3) / NW / a.tiles_n);
  // (never fewer than 64 pixels: the callers' buffers for the sums of a range hold that many ranges)
  a.rows = (int)std::max<long long>(64, (((long long)g.Mrows + want - 1) / want + PX - 1) / PX * PX);
  a.parts = (g.Mrows + a.rows - 1) / a.rows;
  if (p) { p->parts = a.parts; p->rows = a.rows; }
  {
    static const std::string label = std::string("conv1_bf16_") + (MODE == kFwd ? "fwd_" : "bwd_") + std::to_string(KC * 16);
    const double flops = 2.0 * g.Mrows * g.OC * g.IC;
    const double bytes = 2.0 * ((double)g.Mrows * g.IC + (double)g.Mrows * g.OC * (1 + (g.addend ? 1 : 0) + (g.relu_mask ? 1 : 0) + (MODE == kBwd && g.bn_sums ? 1 : 0)) + (double)g.OC * g.IC);
    prof::Scope ps(label.c_str(), flops, bytes, st);
    hipLaunchKernelGGL((conv1_stream_kernel<KC, NW, PX, MODE>), dim3((unsigned)(a.parts * a.tiles_n)), dim3(NW * 64), 0, st, a);
  }
  RESIST_CHECK_LAUNCH("conv1");
  return RESIST_OK;
}

template <int MODE>
int pick(const IgemmArgs &a, hipStream_t st, StatParts *p) {
  return a.IC <= 64 ? launch<4, 4, 64, MODE>(a, st, p) : a.IC <= 128 ? launch<8, 4, 64, MODE>(a, st, p) : launch<16, 4, MODE == kBwd ? 64 : 32, MODE>(a, st, p);
}

}  // namespace

// Up to 256 input channels (their filter rows fill 64 registers); forward without an addend, data gradients without a
// BN whose own ReLU has to be decided again (both would take registers that the kernel does not have).  Few pixels, over which the load of a
// filter of more than 128 channels does not pay, nor of more than 64 before side inputs.  us, igemm_kernel | here, by 2^20 output elements:
//   256 channels, statistics  3.0: 8.1 | 10.0   6.1: 12.6 | 14.6   8.0: 13.6 | 15.1   9.2: 19.3 | 16.6   12.3: 22.4 | 19.4    192 channels  5.7: 11.7 | 12.5   11.5: 18.0 | 16.4
//   128 channels, data gradient with all side inputs  3.1: 9.0 | 9.8   4.0: 9.5 | 10.4   6.1: 16.3 | 15.7    forward, statistics  4.0: 7.5 | 7.7   4.6: 10.9 | 9.7
bool conv1_takes(const IgemmArgs &a, int dt, int mode) {
  const long long out = (long long)a.Mrows * a.OC;
  const bool side = a.addend || a.relu_mask || a.bn_sums;
  if (out < (a.IC > 128 ? 9LL << 20 : a.IC > 64 && mode == kBwd && side ? 6LL << 20 : 0)) return false;
  return dt == DT_BF16 && mode != kEval && a.R == 1 && a.S == 1 && a.stride == 1 && a.pad == 0 && a.IC <= 256 && a.OC >= 128 && a.OC >= 2 * a.IC &&
         !(mode == kBwd ? a.bn_sums && a.bn_self : a.addend != nullptr) && a.Mrows >= 4096;
}

int conv1_launch(const IgemmArgs &a, int mode, hipStream_t st, StatParts *p) {
  return mode == kFwd ? pick<kFwd>(a, st, p) : pick<kBwd>(a, st, p);
}

}  // namespace resist
