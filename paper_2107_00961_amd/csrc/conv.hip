// Implicit-GEMM convolutions on the CDNA4 matrix cores: fp32 (v_mfma_f32_32x32x2_f32) and
// bf16 operands with fp32 accumulation (v_mfma_f32_32x32x16_bf16).
//
// The convolutions of a residual block (the paper's local update, Algorithm 1 inner loop, is an
// ordinary SGD step of the blocks a worker keeps) are computed as GEMMs whose A operand is
// gathered on the fly from the NHWC activation tensor:
//   forward  Y[m=(n,p,q)][k]  = sum_{r,s,c} X[n, p*st+r-pad, q*st+s-pad, c] * W[k][r][s][c]
//   dgrad    dX[m=(n,h,w)][c] = sum_{r,s,k} dY[n, (h+pad-r)/st, (w+pad-s)/st, k] * WT[c][r][s][k]
//            (terms with a non-integer or out-of-range source pixel vanish; for stride 2 the output
//             pixels are processed one parity class at a time so that no such term is ever issued)
//   wgrad    dW[k][r][s][c]   = sum_{m=(n,p,q)} dY[m][k] * X[n, p*st+r-pad, q*st+s-pad, c]
// Tiles are staged through LDS (double buffered, one barrier per K-chunk); every wave owns a
// grid of 32x32 accumulator tiles held in registers.
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "conv_tile.h"

namespace resist {

namespace {

constexpr int kThreads = 256;
#ifndef RESIST_BF16_GLOBAL_DEPTH
#define RESIST_BF16_GLOBAL_DEPTH 2   // chunks an eight-wave bf16 workgroup requests ahead of their use (1..3)
#endif
#ifndef RESIST_BF16_FRAG_DEPTH
#define RESIST_BF16_FRAG_DEPTH 1   // k-steps a bf16 fragment is fetched ahead of its MFMAs (1..3)
#endif
constexpr int kStages = 2;     // LDS double buffering in the implicit-GEMM kernels

// BK: K-chunk (elements) staged per step; LDS rows are padded by 16 bytes (conflict-free b128 reads).
//
// The K loop runs over (filter tap, channel chunk).  Its body is one straight-line block: the
// source pixel of every tile row is (hc + dh, wc + dw) with per-row (hc, wc) fixed for the whole
// kernel and per-tap scalars (dh, dw) kept in scalar registers, loads are hardware-bounds-checked
// buffer loads (an invalid element is requested at an out-of-range offset and comes back as zero),
// and the tap counters are advanced with selects.  With no branch in the loop the scheduler is free
// to place the address arithmetic, the LDS traffic and the global loads in the shadow of the MFMAs.
template <typename T, int BM, int BN, int BK, int WGM, int WGN, int MODE>
__global__ __launch_bounds__(WGM * WGN * 64) void igemm_kernel(ArgsOf<MODE> a) {
  using E = Elem<T>;
  constexpr int NT = WGM * WGN * 64;             // threads: one wave per wave tile, 4 or 8 waves
  constexpr int VEC = E::VEC;
  constexpr int ES = (int)sizeof(T);
  constexpr int LDK = BK + VEC;
  constexpr int WTM = BM / WGM, WTN = BN / WGN;  // wave tile
  constexpr int TM = WTM / 32, TN = WTN / 32;    // 32x32 MFMA tiles per wave
  constexpr int KV = BK / VEC;                   // lanes per tile row (16 bytes each)
  constexpr int RPP = NT / KV;             // tile rows per load pass
  constexpr int PA = BM / RPP, PB = BN / RPP;    // load passes
  constexpr int NK = BK / (2 * VEC);             // k-steps per chunk
  static_assert((WGM * WGN == 4 || WGM * WGN == 8) && TM >= 1 && TN >= 1 && PA >= 1 && PB >= 1 && NK >= 2, "tile shape");
  // one LDS block: the operand stages during the K loop, the fp32 output tile afterwards
  constexpr int LDC = BN + 8;   // output tile pitch (floats): lanes l and l+32 (4 rows apart) hit disjoint banks
  constexpr size_t kOperandBytes = sizeof(T) * kStages * (BM + BN) * LDK;
  constexpr size_t kTileBytes = sizeof(float) * BM * LDC;
  static_assert(kTileBytes <= kOperandBytes, "output tile must fit in the operand stages");
  __shared__ __attribute__((aligned(16))) char lds_raw[kOperandBytes];
  T (*As)[BM][LDK] = reinterpret_cast<T (*)[BM][LDK]>(lds_raw);
  T (*Bs)[BN][LDK] = reinterpret_cast<T (*)[BN][LDK]>(lds_raw + sizeof(T) * kStages * BM * LDK);
  float (*Cs)[LDC] = reinterpret_cast<float (*)[LDC]>(lds_raw);
  __shared__ int row_off[BM];

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WGN, wn = wave % WGN;

  // Logical tile order: N-tiles fastest, so tiles sharing input rows are neighbours; each XCD gets a
  // contiguous range of them.  The stride-2 data gradient (4 parity classes of unequal work, class
  // slowest) keeps the hardware round-robin order, which measured faster for its short K loops.
  int bid = a.cls == 1 ? xcd_contiguous(blockIdx.x, gridDim.x) : (int)blockIdx.x;
  const int bq = fdiv(bid, a.div_tn);
  const int tn = bid - bq * a.tiles_n;
  const int cidx = fdiv(bq, a.div_tm);   // parity class
  const int tm = bq - cidx * a.tiles_m;
  const int ph = a.cls == 2 ? cidx >> 1 : 0, pw = a.cls == 2 ? cidx & 1 : 0;   // cls is 1 or 2
  const int m0 = tm * BM, n0 = tn * BN;

  // filter taps that contribute: r = r0, r0+tstep, ... < R (all taps unless MODE==kBwd, stride 2)
  int r0 = 0, s0 = 0, tstep = 1;
  if (MODE == kBwd && a.stride == 2) { r0 = (ph + a.pad) & 1; s0 = (pw + a.pad) & 1; tstep = 2; }
  const int nr = r0 < a.R ? (tstep == 2 ? (a.R - r0 + 1) >> 1 : a.R - r0) : 0;
  const int ns = s0 < a.S ? (tstep == 2 ? (a.S - s0 + 1) >> 1 : a.S - s0) : 0;
  const int cchunks = (a.IC + BK - 1) / BK;
  const int nchunks = nr * ns * cchunks;

  // per-thread tile rows: centre pixel (hc, wc) and byte offset of its first channel of interest
  const int lrow = tid / KV, kvec = (tid % KV) * VEC;
  int hc[PA], wc[PA], aoff[PA], boff[PB];
#pragma unroll
  for (int i = 0; i < PA; ++i) {
    const int m = m0 + i * RPP + lrow;
    if (m < a.Mrows) {
      const int n = fdiv(m, a.div_plane);
      const int rem = m - n * (a.OHc * a.OWc);
      const int ohc = fdiv(rem, a.div_w), owc = rem - ohc * a.OWc;
      if (MODE != kBwd) { hc[i] = ohc * a.stride - a.pad; wc[i] = owc * a.stride - a.pad; }
      else if (a.stride == 1) { hc[i] = ohc + a.pad; wc[i] = owc + a.pad; }
      else { hc[i] = ohc; wc[i] = owc; }
      aoff[i] = (((n * a.IH + hc[i]) * a.IW + wc[i]) * a.IC + kvec) * ES;
    } else {
      hc[i] = -(1 << 24); wc[i] = -(1 << 24); aoff[i] = 0;   // never in range
    }
  }
#pragma unroll
  for (int i = 0; i < PB; ++i) {
    const int oc = n0 + i * RPP + lrow;
    boff[i] = oc < a.OC ? (oc * a.R * a.S * a.IC + kvec) * ES : (int)kOOB;
  }
  for (int r = tid; r < BM; r += NT) {
    const int m = m0 + r;
    int off = -1;
    if (m < a.Mrows) {
      const int n = fdiv(m, a.div_plane);
      const int rem = m - n * (a.OHc * a.OWc);
      const int orow = fdiv(rem, a.div_w);
      const int oh = orow * a.cls + ph, ow = (rem - orow * a.OWc) * a.cls + pw;
      off = (n * a.OH + oh) * a.OW + ow;
    }
    row_off[r] = off;
  }

  const __amdgpu_buffer_rsrc_t rin = make_rsrc(a.in, (unsigned)a.N * a.IH * a.IW * a.IC * ES);
  const __amdgpu_buffer_rsrc_t rwt = make_rsrc(a.wt, (unsigned)a.OC * a.R * a.S * a.IC * ES);

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  // loop state of the chunk that will be requested next (uniform across the workgroup)
  int tr = r0, ts = s0, tc = 0, issued = 0;
  // GD = how many chunks ahead of its use an operand chunk is requested from global memory (GD
  // register sets in a ring).  An eight-wave workgroup is alone on its CU, so no other workgroup
  // covers the latency of its loads, and a bf16 chunk is multiplied in less time than a load takes.
  constexpr int GD = (ES == 2 && NT == 512) ? RESIST_BF16_GLOBAL_DEPTH : 1;
  f32x4 ra[GD][PA], rb[GD][PB];
  // scalars of the chunk being requested (set by begin_chunk, used by request)
  int q_dh = 0, q_dw = 0, q_adelta = 0, q_bdelta = 0;
  bool q_kok = false;
  auto begin_chunk = [&]() {
    // tap scalars: source pixel displacement and the byte deltas of activation and filter
    if (MODE != kBwd) { q_dh = tr; q_dw = ts; }
    else if (a.stride == 1) { q_dh = -tr; q_dw = -ts; }
    else { q_dh = (ph + a.pad - tr) >> 1; q_dw = (pw + a.pad - ts) >> 1; }   // even by construction
    const bool live = issued < nchunks;
    const int c0 = tc * BK;
    q_adelta = ((q_dh * a.IW + q_dw) * a.IC + c0) * ES;
    q_bdelta = ((tr * a.S + ts) * a.IC + c0) * ES;
    q_kok = live && (c0 + kvec) < a.IC;
    // advance (tap, channel chunk) without branches
    ++issued;
    const bool cwrap = (tc + 1 == cchunks);
    tc = cwrap ? 0 : tc + 1;
    const bool swrap = cwrap && (ts + tstep >= a.S);
    ts = cwrap ? (swrap ? s0 : ts + tstep) : ts;
    tr = swrap ? tr + tstep : tr;
  };
  // register `part` (0..PA-1: activation rows, PA..PA+PB-1: filter rows) of the chunk begun last
  auto request = [&](int set, int part) {
    if (part < PA) {
      const int i = part;
      const bool ok = q_kok && (unsigned)(hc[i] + q_dh) < (unsigned)a.IH && (unsigned)(wc[i] + q_dw) < (unsigned)a.IW;
      ra[set][i] = buffer_load_16B(rin, ok ? (unsigned)(aoff[i] + q_adelta) : kOOB);
    } else {
      const int i = part - PA;
      rb[set][i] = buffer_load_16B(rwt, q_kok ? (unsigned)(boff[i] + q_bdelta) : kOOB);
    }
  };
  auto store_part = [&](int set, int stage, int part) {
    if (part < PA) *reinterpret_cast<f32x4 *>(&As[stage][part * RPP + lrow][kvec]) = ra[set][part];
    else *reinterpret_cast<f32x4 *>(&Bs[stage][(part - PA) * RPP + lrow][kvec]) = rb[set][part - PA];
  };
  auto load_global = [&](int set) {
    begin_chunk();
#pragma unroll
    for (int p = 0; p < PA + PB; ++p) request(set, p);
  };
  auto store_lds = [&](int set, int stage) {
#pragma unroll
    for (int p = 0; p < PA + PB; ++p) store_part(set, stage, p);
  };

  // Pipeline.  Chunk `it` is multiplied out of LDS stage it&1, one k-step (2*VEC values of K) at a
  // time; the fragments of a k-step are fetched from LDS during the MFMAs of the k-step before it,
  // also across the chunk boundary.  The registers holding chunk it+1 (requested from global memory
  // one chunk of MFMA time earlier) go to the other stage, and chunk it+2 is requested into them,
  // a few registers per k-step over k-steps 0 .. NK-FD-1, so that neither the LDS nor the memory
  // pipeline sees a burst.  The one barrier per chunk sits at the start of the first k-step whose
  // fetch reaches into the next chunk: by then every wave has all fragments of this stage in
  // registers and has written its share of the next stage, so after it the first fragments of chunk
  // it+1 can be fetched while the last MFMAs run.
  // FD = how many k-steps ahead of its MFMAs a fragment is fetched; NB fragment buffers in a ring.
  // The bf16 matrix instruction runs 32 cycles and every MFMA of a 32x32 wave tile depends on the one
  // before it, so one k-step ahead leaves a wave waiting on the LDS for most of each step.
  constexpr int FD = (ES == 2 && NK % 4 == 0) ? RESIST_BF16_FRAG_DEPTH : 1;
  constexpr int NB = FD == 1 ? 2 : 4;
  static_assert(NK % NB == 0 && FD >= 1 && FD < NB && FD < NK, "fragment ring");
  const int lr = lane & 31, lk = (lane >> 5) * VEC;
  f32x4 fa[NB][TM], fb[NB][TN];
  auto load_frags = [&](int buf, int stage, int ks) {
#pragma unroll
    for (int i = 0; i < TM; ++i) fa[buf][i] = *reinterpret_cast<const f32x4 *>(&As[stage][wm * WTM + i * 32 + lr][ks * 2 * VEC + lk]);
#pragma unroll
    for (int j = 0; j < TN; ++j) fb[buf][j] = *reinterpret_cast<const f32x4 *>(&Bs[stage][wn * WTN + j * 32 + lr][ks * 2 * VEC + lk]);
  };
  auto lds_barrier = [&]() {
    __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0): this wave's LDS writes and reads are done
    __builtin_amdgcn_s_barrier();
  };

  load_global(0);
  store_lds(0, 0);
#pragma unroll
  for (int c = 1; c <= GD; ++c) load_global(c % GD);   // chunk c waits in register set c % GD
  lds_barrier();
#pragma unroll
  for (int d = 0; d < FD; ++d) load_frags(d, 0, d);
  __builtin_amdgcn_sched_barrier(0);

  // chunk `it`: multiplied out of its stage while chunk it+1 moves from register set `set` to the other
  // stage and chunk it+1+GD is requested into that set
  auto chunk_body = [&](int set, int stage) {
#pragma unroll
    for (int ks = 0; ks < NK; ++ks) {
      const int kn = ks + FD;              // the k-step whose fragments are fetched now
      if (kn < NK) {
        load_frags(kn % NB, stage, kn);
      } else {
        if (kn == NK) lds_barrier();       // once per chunk, at the start of k-step NK-FD
        load_frags(kn % NB, stage ^ 1, kn - NK);   // past the last chunk: zeros nobody uses
      }
      __builtin_amdgcn_sched_barrier(0);   // keep the fetches ahead of this k-step's MFMAs
      if (ks == 0) begin_chunk();
#pragma unroll
      for (int p = 0; p < PA + PB; ++p)
        if ((p * (NK - FD)) / (PA + PB) == ks) {   // parts spread evenly over k-steps 0 .. NK-FD-1
          store_part(set, stage ^ 1, p);
          request(set, p);
        }
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) E::mma(acc[i][j], fa[ks % NB][i], fb[ks % NB][j]);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  for (int it = 0; it < nchunks; it += GD) {
#pragma unroll
    for (int j = 0; j < GD; ++j) {
      if (j > 0 && it + j >= nchunks) break;   // uniform across the workgroup
      chunk_body((j + 1) % GD, (it + j) & 1);
    }
  }

  // A lane holds column (lane%32) and rows 8*(e/4) + 4*(lane/32) + e%4 of each 32x32 tile.  The operand stages are
  // free after the last barrier (every fragment a wave uses was fetched before it) and take the output tile.
  conv_epilogue<T, BM, BN, NT, MODE>(a, Cs, row_off, tm, n0, [&]() {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int cl = wn * WTN + j * 32 + lr;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int row = wm * WTM + i * 32 + (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3);
          Cs[row][cl] = acc[i][j][e];
        }
      }
  });
}

template <typename T, int BM, int BN, int BK, int WGM, int WGN, int MODE>
int launch_igemm(EvalArgs a, hipStream_t st, StatParts *tiles_m_out) {
  a.tiles_m = (a.Mrows + BM - 1) / BM;
  if (tiles_m_out) { tiles_m_out->parts = a.tiles_m; tiles_m_out->rows = BM; }
  a.tiles_n = (a.OC + BN - 1) / BN;
  a.div_plane = make_fastdiv((unsigned)(a.OHc * a.OWc)); a.div_w = make_fastdiv((unsigned)a.OWc);
  a.div_tn = make_fastdiv((unsigned)a.tiles_n); a.div_tm = make_fastdiv((unsigned)a.tiles_m);
  const long long grid = (long long)a.tiles_m * a.tiles_n * a.cls * a.cls;
  if (grid <= 0 || grid > 0x7fffffffLL) return set_error(RESIST_ESHAPE, "igemm grid %lld", grid);
  {
    static const std::string label = std::string("igemm_") + (sizeof(T) == 4 ? "f32_" : "bf16_") + (MODE == kFwd ? "fwd_" : MODE == kEval ? "eval_" : "bwd_") +
                                     std::to_string(BM) + "x" + std::to_string(BN) + "x" + std::to_string(BK) +
                                     (WGM * WGN == 8 ? "_w8" : "");
    // algorithmic work of the convolution this launch computes (forward or data gradient)
    const double flops = 2.0 * a.N * (MODE != kBwd ? (double)a.OH * a.OW : (double)a.IH * a.IW) * a.OC * a.IC * a.R * a.S;
    const double bytes = sizeof(T) * ((double)a.N * a.IH * a.IW * a.IC + (double)a.N * a.OH * a.OW * a.OC * (1 + (a.addend ? 1 : 0) + (a.relu_mask ? 1 : 0) + (MODE == kBwd && a.bn_sums ? 1 : 0) +
                                       (MODE == kEval ? (a.out ? 1 : 0) + (a.act_res ? 1 : 0) : 0)) +
                                      (double)a.OC * a.R * a.S * a.IC);
    prof::Scope ps(label.c_str(), flops, bytes, st);
    hipLaunchKernelGGL((igemm_kernel<T, BM, BN, BK, WGM, WGN, MODE>), dim3((unsigned)grid), dim3(WGM * WGN * 64), 0, st, static_cast<const ArgsOf<MODE> &>(a));
  }
  RESIST_CHECK_LAUNCH("igemm");
  return RESIST_OK;
}

template <typename T, int MODE>
int dispatch_igemm(const EvalArgs &a, hipStream_t st, StatParts *tiles_m_out = nullptr) {
  constexpr int dt = sizeof(T) == 2 ? DT_BF16 : DT_F32;
  if (conv_small_takes(a, dt)) return conv_small_launch(a, dt, MODE, st, tiles_m_out);
  if constexpr (sizeof(T) == 4 && MODE != kEval) {   // (the test-time forward prepares its filters)
    if (conv3_takes(a, dt)) return conv3_launch_rows(a, MODE, st, tiles_m_out);
  }
  if (conv1_takes(a, dt, MODE)) return conv1_launch(a, MODE, st, tiles_m_out);
  // pick the largest tile that still yields enough workgroups to cover the 256 compute units
  constexpr int V = Elem<T>::VEC;   // K-chunks of 8*V and 16*V elements: 128 and 256 bytes per tile row
  const long long classes = (long long)a.cls * a.cls;
  auto tiles = [&](int bm, int bn) {
    return (long long)((a.Mrows + bm - 1) / bm) * ((a.OC + bn - 1) / bn) * classes;
  };
  constexpr long long kMin = 512;
  constexpr bool lp = sizeof(T) == 2;
  // fp32 is bound by the matrix cores, and 64x64 tiles with little LDS, several to a compute unit, keep them busiest; up to two to a unit the
  // longer chunk is the faster.  us, 128x128 | 128x64 | 64x64 in chunks of 64 | of 32 channels: 128 -> 128 ch 1x1, 33280 pixels 27.3 | 25.6 |
  // 22.8 | 21.5, 16000 pixels 18.1 | 13.0 | 12.1 | 12.3; 64 -> 128 ch 3x3 stride 2, 102400 pixels 158.9 | 149.4 | 142.8 | 133.4, its data
  // gradient from 32768 127 | 73.5 | 67.2 | 60.1.  (Before: 128x128 from 512 tiles, then 128x64.)
  if constexpr (!lp) {
    // (the test-time forward: 128x128 from 512 tiles, as it is tested)
    if (MODE == kEval && a.OC > 64 && tiles(128, 128) >= kMin) return launch_igemm<T, 128, 128, 8 * V, 2, 2, MODE>(a, st, tiles_m_out);
    if (a.IC % (16 * V) == 0 && tiles(64, 64) <= 512) return launch_igemm<T, 64, 64, 16 * V, 2, 2, MODE>(a, st, tiles_m_out);
    return launch_igemm<T, 64, 64, 8 * V, 2, 2, MODE>(a, st, tiles_m_out);
  } else {
    const long long t128 = tiles(128, 128), t64 = tiles(128, 64);
    const bool deep = a.IC % (16 * V) == 0;
    if constexpr (MODE != kFwd) {
      // The test-time forward, in the tiles that its epilogue is tested in (those of the model below measure faster where these fill their last
      // round badly, 128 ch 28x28 3x3, batch 31 22.8 | 17.9 us, 64 -> 192 ch 56x56 1x1, batch 64 70.8 | 60.1), and the parity classes of strided data
      // gradients: the 128x128 tile moves half the operand bytes per FLOP; of eight waves where there is about one to a compute unit
      // (256 -> 256 ch 14x14, batch 64 29.0 -> 24.1 us), or 128x64 where there are fewer.
      if (MODE == kEval || a.cls != 1) {
        if (MODE == kEval && a.OC >= 128) {
          if (t128 >= 192 && t128 < 320) return launch_igemm<T, 128, 128, 8 * V, 4, 2, MODE>(a, st, tiles_m_out);
          if (t128 < 192 && t64 >= 256 && deep) return launch_igemm<T, 128, 64, 16 * V, 4, 2, MODE>(a, st, tiles_m_out);
        }
        if (a.OC > 64 && t128 >= 192) return launch_igemm<T, 128, 128, 8 * V, 2, 2, MODE>(a, st, tiles_m_out);
        if (MODE == kEval && a.OC <= 64 && t64 >= kMin) return launch_igemm<T, 128, 64, 8 * V, 4, 2, MODE>(a, st, tiles_m_out);
        if (t64 >= kMin) return launch_igemm<T, 128, 64, 8 * V, 2, 2, MODE>(a, st, tiles_m_out);
        if (deep) return launch_igemm<T, 64, 64, 16 * V, 2, 2, MODE>(a, st, tiles_m_out);
        return launch_igemm<T, 64, 64, 8 * V, 2, 2, MODE>(a, st, tiles_m_out);
      }
    }
    // bf16: the tile with the least time by a model of it, us: a launch's start and end, and for every workgroup that the fullest of the 256
    // compute units gets a constant and a part per reduction index (IC*R*S).  An area of 128x128 costs about the same in all of them, a third
    // more in 64x64, so what counts is how the last round fills the chip.  Measured, us, 128x128 of eight waves | of four | 128x64 | 64x64:
    //   128 -> 128 ch 3x3, 110 tiles of 128x128 16.7 | 20.0 | 13.6 | 14.4    180: 17.0 | 20.9 | 19.2 | 17.8    270: 29.1 | 26.4 | 25.6 | 25.4
    //                                       500 30.5 | 29.5 | 33.2 | 36.7    900: 54.7 | 50.9 | 63.8 | 61.3
    //   256 -> 128 ch 1x1, 140: 10.1 | 11.2 | 9.8 | 10.0    270: 15.4 | 14.1 | 13.2 | 12.8    400: 15.4 | 15.0 | 15.4 | 15.1
    //   192 -> 320 ch 1x1, 270: 13.4 | 12.4 | 9.6 | 10.6    64 -> 64 ch 3x3, 180 tiles of 128x64: -- | -- | 9.6 | 10.1    270: -- | -- | 13.5 | 11.6
    // It is right to a tenth, so it is asked for what it gains over the tile by the number of tiles alone: 128x128 of eight waves from 192 to
    // 319 tiles, of four from there up, 128x64 in chunks of 128 channels from 256 of them (whose second workgroup a compute unit does not hold
    // beside the first).  Where BN sums are taken, smaller tiles pay for them more often: 128x128 is left for a tenth or more.  us, 128x128 |
    // smaller, predicted: 256 -> 1024 ch 14x14, batch 31, statistics 12.6 | 14.0, 0.99; data gradient to 192 ch 56x56 from 384 with all its
    // side inputs 51.0 | 56.2, 0.96; from 64 -> 192 ch without sums 41.2 | 30.7, 0.86.  And 128x64 for 64x64, without sums, for a fortieth:
    // 256 -> 64 ch 56x56, batch 128 41.4 | 43.7, 0.99; with sums, for a reduction of no whole 128 channels, 128x64 for 64x64 for a tenth: data gradient
    // to 64 ch 56x56 from 192, batch 16 10.7 | 10.2, 0.95.
    const double k = (double)a.IC * a.R * a.S;
    auto rounds = [](long long n) { return (double)((n + 255) / 256); };
    const double r128 = rounds(t128), r64 = rounds(t64), r32 = rounds(tiles(64, 64));
    enum { kEight, kFour, kHalf, kQuarter };
    const double cost[] = {5 + r128 * (3.5 + 7.8e-3 * k), 5 + r128 * (r128 == 1 ? 1.3 : 1.0) * (2.8 + 7.3e-3 * k), 5.3 + r64 * (1.8 + 4.5e-3 * k),
                           6 + r32 * (0.75 + 2.9e-3 * k)};
    const int usual = a.OC > 64 && t128 >= 192 ? (a.OC >= 128 && t128 < 320 ? kEight : kFour)
                                               : t64 >= kMin || (a.OC >= 128 && t64 >= 256 && deep) ? kHalf : kQuarter;
    int best = (int)(std::min_element(cost + (a.OC > 64 ? kEight : kHalf), cost + 4) - cost);
    const bool sums = a.stats || a.bn_sums;
    const double worth = sums && (usual <= kFour ? best >= kHalf : usual == kQuarter && !deep) ? 0.9 : !sums && usual == kHalf && best == kQuarter ? 0.975 : 1.0;
    if (cost[best] > worth * cost[usual]) best = usual;
    // chunks of 128 channels where a unit gets one workgroup (two of 64x64) and the reduction is long
    if (best == kEight) return launch_igemm<T, 128, 128, 8 * V, 4, 2, MODE>(a, st, tiles_m_out);
    if (best == kFour) return launch_igemm<T, 128, 128, 8 * V, 2, 2, MODE>(a, st, tiles_m_out);
    if (best == kHalf)
      return deep && r64 == 1 && k >= 1024 ? launch_igemm<T, 128, 64, 16 * V, 4, 2, MODE>(a, st, tiles_m_out) : launch_igemm<T, 128, 64, 8 * V, 4, 2, MODE>(a, st, tiles_m_out);
    return deep && (r32 == 1 || (r32 == 2 && k >= 1024)) ? launch_igemm<T, 64, 64, 16 * V, 2, 2, MODE>(a, st, tiles_m_out)
                                                         : launch_igemm<T, 64, 64, 8 * V, 2, 2, MODE>(a, st, tiles_m_out);
  }
}

int check_geom(const ConvGeom &g, int dt) {
  const int v = dt == DT_BF16 ? 8 : 4;
  if (dt != DT_F32 && dt != DT_BF16) return set_error(RESIST_EINVAL, "dtype %d", dt);
  if (g.N < 1 || g.H < 1 || g.W < 1 || g.C < v || g.K < v || (g.C % v) || (g.K % v))
    return set_error(RESIST_ESHAPE, "conv shape N%d H%d W%d C%d K%d (C, K must be multiples of %d)", g.N, g.H, g.W, g.C, g.K, v);
  if (g.R != g.S || (g.R != 1 && g.R != 3 && g.R != 5 && g.R != 7))
    return set_error(RESIST_ESHAPE, "filter %dx%d unsupported", g.R, g.S);
  if (g.stride < 1 || g.stride > 2 || g.pad < 0 || g.pad >= g.R)
    return set_error(RESIST_ESHAPE, "stride %d pad %d unsupported", g.stride, g.pad);
  if (g.P < 1 || g.Q < 1) return set_error(RESIST_ESHAPE, "empty convolution output");
  const long long lim = 0x7fffffffLL / (dt == DT_BF16 ? 2 : 4);   // byte offsets stay below the out-of-range marker
  if ((long long)g.N * g.H * g.W * g.C > lim || (long long)g.N * g.P * g.Q * g.K > lim ||
      (long long)g.K * g.R * g.S * g.C > lim)
    return set_error(RESIST_ESHAPE, "tensor exceeds 2 GiB");
  return RESIST_OK;
}

}  // namespace

int conv_check(const ConvGeom &g, int dt) { return check_geom(g, dt); }

bool filter_in_fragments(const ConvGeom &g, int dt, bool dgrad) {
  if (g.R != 3 || g.S != 3 || g.stride != 1 || g.pad != 1 || (int64_t)g.N * g.H * g.W > 0x7fffffff) return false;
  IgemmArgs a{};
  a.N = g.N; a.IH = a.OH = a.OHc = g.H; a.IW = a.OW = a.OWc = g.W;
  a.IC = dgrad ? g.K : g.C; a.OC = dgrad ? g.C : g.K;
  a.R = a.S = 3; a.stride = a.pad = a.cls = 1;
  a.Mrows = g.N * g.H * g.W;
  return conv3_takes(a, dt) && !conv_small_takes(a, dt);
}

int64_t filter_bytes(const ConvGeom &g, int dt, bool fragments, bool dgrad) {
  if (!fragments) return (int64_t)g.K * g.R * g.S * g.C * esize(dt);
  return conv3_filter_bytes(dgrad ? g.C : g.K, dgrad ? g.K : g.C, dt);
}

int64_t conv_stats_floats(const ConvGeom &g) {
  // the smallest row tile a forward kernel uses is 64, of a small output 32
  const int64_t M = (int64_t)g.N * g.P * g.Q, rows = conv_small_rows(M, g.K, 1) ? 32 : 64;
  return 3 * ((M + rows - 1) / rows) * g.K;
}

int conv_fwd(const ConvGeom &g, int dt, const void *x, const Filter &w, void *y, const void *addend, float *stats, StatParts *stat_parts,
             hipStream_t st, const EvalAct *act) {
  RESIST_TRY(check_geom(g, dt));
  if (stats && !stat_parts) return set_error(RESIST_EINVAL, "conv_fwd: stats without stat_parts");
  EvalArgs a{};
  a.in = x; a.wt = w.fragments || !w.prep ? w.w : w.prep; a.out = y; a.addend = addend; a.stats = stats;
  if (!a.wt && !w.fragments) return set_error(RESIST_EINVAL, "conv_fwd: no filter");
  a.N = g.N; a.IH = g.H; a.IW = g.W; a.IC = g.C;
  a.OH = g.P; a.OW = g.Q; a.OC = g.K;
  a.R = g.R; a.S = g.S; a.stride = g.stride; a.pad = g.pad;
  a.cls = 1; a.OHc = g.P; a.OWc = g.Q;
  a.Mrows = g.N * g.P * g.Q;
  if (act) {
    if (stats || !act->out || !act->scale || !act->shift) return set_error(RESIST_EINVAL, "conv_fwd: fused activation");
    a.act = act->out; a.act_scale = act->scale; a.act_shift = act->shift;
    a.act_res = act->res; a.res_scale = act->rscale; a.res_shift = act->rshift;
    if (w.fragments) return conv3_launch(a, w, dt, kEval, st, nullptr);
    return dt == DT_BF16 ? dispatch_igemm<__bf16, kEval>(a, st) : dispatch_igemm<float, kEval>(a, st);
  }
  if (w.fragments) return conv3_launch(a, w, dt, kFwd, st, stat_parts);
  return dt == DT_BF16 ? dispatch_igemm<__bf16, kFwd>(a, st, stat_parts) : dispatch_igemm<float, kFwd>(a, st, stat_parts);
}

int conv_dgrad(const ConvGeom &g, int dt, const void *dy, const Filter &w, void *dx, const void *addend, const void *relu_mask,
               hipStream_t st, const BnBwdFuse *bn) {
  RESIST_TRY(check_geom(g, dt));
  if (g.stride == 2 && ((g.H & 1) || (g.W & 1)))
    return set_error(RESIST_ESHAPE, "stride-2 dgrad needs even input size, got %dx%d", g.H, g.W);
  EvalArgs a{};
  if (!w.prep) return set_error(RESIST_EINVAL, "conv_dgrad: no prepared filter");
  a.in = dy; a.wt = w.fragments ? w.w : w.prep; a.out = dx; a.addend = addend; a.relu_mask = relu_mask;
  a.N = g.N; a.IH = g.P; a.IW = g.Q; a.IC = g.K;
  a.OH = g.H; a.OW = g.W; a.OC = g.C;
  a.R = g.R; a.S = g.S; a.stride = g.stride; a.pad = g.pad;
  a.cls = g.stride; a.OHc = g.H / g.stride; a.OWc = g.W / g.stride;
  a.Mrows = g.N * a.OHc * a.OWc;
  StatParts parts;
  if (bn) {
    if (a.cls != 1 || !bn->y || !bn->sums || !bn->parts) return set_error(RESIST_EINVAL, "fused BN sums need a stride-1 data gradient");
    a.bn_y = bn->y; a.bn_mean = bn->b.mean; a.bn_invstd = bn->b.invstd; a.bn_scale = bn->b.scale; a.bn_shift = bn->b.shift;
    a.bn_sums = bn->sums; a.bn_self = bn->relu_of_self ? 1 : 0;
  }
  if (w.fragments) RESIST_TRY(conv3_launch(a, w, dt, kBwd, st, &parts));
  else RESIST_TRY(dt == DT_BF16 ? (dispatch_igemm<__bf16, kBwd>(a, st, &parts)) : (dispatch_igemm<float, kBwd>(a, st, &parts)));
  if (bn) *bn->parts = parts;
  return RESIST_OK;
}

int64_t conv_dgrad_bn_sums_floats(const ConvGeom &g) {
  // the smallest row tile a data-gradient kernel uses is 64, of a small output 32
  const int64_t M = (int64_t)g.N * g.H * g.W, rows = conv_small_rows(M, g.C, 1) ? 32 : 64;
  return 2 * ((M + rows - 1) / rows) * g.C;
}

// ---- filter preparation ------------------------------------------------------------------------------
// All filters of a step in one launch (or a few: the table travels in the kernel arguments).
namespace {
constexpr int kPrepSegs = 48;
// (a table of one for a single filter: shorter arguments and no search, 3.5 instead of 4.1 us for 256x80x3x3 in bf16)
template <int N> struct PrepTable {
  const void *w[N];
  void *wlp[N];
  void *wT[N];
  int K[N], RS[N], C[N];
  float scale[N];
  int first_wg[N + 1];
  unsigned long long frag_copy, frag_transpose;   // bit per filter: in matrix fragments (conv3.hip) instead of rows
  int nseg;
};
// (a caller's filter or workspace need not be aligned to more than its elements)
typedef f32x4 __attribute__((aligned(4))) f32x4_any;
typedef u32x2 __attribute__((aligned(2))) u32x2_any;
__device__ inline f32x4 load4(const float *p) { return *reinterpret_cast<const f32x4_any *>(p); }
__device__ inline f32x4 load4(const __bf16 *p) {
  const u32x2 t = *reinterpret_cast<const u32x2_any *>(p);
  return f32x4{bf16_lo(t[0]), bf16_hi(t[0]), bf16_lo(t[1]), bf16_hi(t[1])};
}
// four consecutive elements of T from four floats
__device__ inline void store4(float *p, float a, float b, float c, float d) {
  *reinterpret_cast<f32x4_any *>(p) = f32x4{a, b, c, d};
}
__device__ inline void store4(__bf16 *p, float a, float b, float c, float d) {
  *reinterpret_cast<u32x2_any *>(p) = u32x2{pack_bf16x2(a, b), pack_bf16x2(c, d)};
}

// 64 output channels x 64 input channels of one tap, at(oc, ch), as the fragments that conv3.hip multiplies with: its layout is
// [octile of 32][chunk of 64 channels][tap][slice of 16][part][lane][8 values], lane l holding output channel l % 32 and channels
// 8 * (l / 32) .. +7 of its slice; fp32 in three bf16 parts.  Behind them one word per 64x64 tile and tap, [tile][chunk][tap]:
// whether it holds a value that three parts do not.
template <typename T, typename At>
__device__ inline void store_fragments(void *out, int octiles, int chunks, int octile, int chunk, int tap, At at) {
  constexpr int NP = sizeof(T) == 4 ? 3 : 1;
  unsigned long long missed = 0;
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int id = threadIdx.x + u * 256;          // (half, slice, lane)
    const int lane = id & 63, slice = (id >> 6) & 3, half = id >> 8;
    const int oc = half * 32 + (lane & 31), ch = slice * 16 + (lane >> 5) * 8;
    f32x4 lo, hi;
#pragma unroll
    for (int e = 0; e < 4; ++e) { lo[e] = at(oc, ch + e); hi[e] = at(oc, ch + 4 + e); }
    char *dst = static_cast<char *>(out) + ((((size_t)(octile * 2 + half) * chunks + chunk) * 9 + tap) * 4 + slice) * (NP * 1024) + lane * 16;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      if (NP == 3 && p == 2) { split_check(lo, missed); split_check(hi, missed); }
      const u32x2 a = split_part(lo), b = split_part(hi);
      *reinterpret_cast<u32x4 *>(dst + p * 1024) = u32x4{a[0], a[1], b[0], b[1]};
    }
  }
  if constexpr (NP == 3) {
    const int any = __syncthreads_or(missed != 0);
    unsigned *flags = reinterpret_cast<unsigned *>(static_cast<char *>(out) + (size_t)octiles * 2 * chunks * 9 * 4 * (NP * 1024));
    if (threadIdx.x == 0) flags[((size_t)octile * chunks + chunk) * 9 + tap] = any ? 1u : 0u;
  }
}

// One 64x64 tile of the [K][C] matrix of one tap per workgroup, through LDS so that both sides move whole
// vectors: 256-byte runs of the fp32 master in, 4-element vectors of the copy and of the transpose out.  A single filter that is
// not wanted in fragments is a matter of latency, and taken in 32x32 tiles (data gradients of small 1x1 layers, with the preparation, us,
// 64x64 -> 32x32: bf16 256 from 512 ch 14x14, batch 8 9.2 -> 8.3, fp32 128 from 64 ch 16x16, batch 64 11.8 -> 10.8).
template <typename S, typename T, int N, int TS>
__global__ __launch_bounds__(256) void prepare_filters_kernel(PrepTable<N> t) {
  constexpr int kVecs = TS / 4, kRows = 256 / kVecs, kPasses = TS / kRows;
  __shared__ float tile[TS][TS + 1];
  int seg = 0;
  while (N > 1 && seg + 1 < t.nseg && (int)blockIdx.x >= t.first_wg[seg + 1]) ++seg;
  const int K = t.K[seg], RS = t.RS[seg], C = t.C[seg];
  int ct, kt, c0, k0, tap;
  if constexpr (N == 1) {
    ct = gridDim.x; kt = gridDim.y;
    c0 = blockIdx.x * TS; k0 = blockIdx.y * TS; tap = blockIdx.z;
  } else {
    ct = (C + TS - 1) / TS; kt = (K + TS - 1) / TS;
    int id = blockIdx.x - t.first_wg[seg];
    c0 = (id % ct) * TS;
    id /= ct;
    k0 = (id % kt) * TS; tap = id / kt;
  }
  const S *__restrict__ w = static_cast<const S *>(t.w[seg]);
  const float sc = t.scale[seg];
  const bool frag_copy = (t.frag_copy >> seg) & 1, frag_transpose = (t.frag_transpose >> seg) & 1;
  T *__restrict__ wlp = static_cast<T *>(t.wlp[seg]);
  T *__restrict__ wT = static_cast<T *>(t.wT[seg]);
  const int row = threadIdx.x / kVecs, col = (threadIdx.x % kVecs) * 4;   // kRows rows x kVecs vectors per pass
  // K and C are multiples of four (checked on the host)
  f32x4 v[kPasses];
#pragma unroll
  for (int p = 0; p < kPasses; ++p) {
    const int k = k0 + row + kRows * p, c = c0 + col;
    v[p] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (k < K && c < C) v[p] = load4(w + ((size_t)k * RS + tap) * C + c);
  }
#pragma unroll
  for (int p = 0; p < kPasses; ++p) {
    const int k = k0 + row + kRows * p, c = c0 + col;
    v[p] *= sc;
    if (wlp && !frag_copy && k < K && c < C) store4(wlp + ((size_t)k * RS + tap) * C + c, v[p][0], v[p][1], v[p][2], v[p][3]);
#pragma unroll
    for (int e = 0; e < 4; ++e) tile[row + kRows * p][col + e] = v[p][e];
  }
  __syncthreads();
  if constexpr (TS == 64) {
    if (wlp && frag_copy) store_fragments<T>(wlp, kt, ct, k0 / TS, c0 / TS, tap, [&](int oc, int ch) { return tile[oc][ch]; });
    if (wT && frag_transpose) store_fragments<T>(wT, ct, kt, c0 / TS, k0 / TS, tap, [&](int oc, int ch) { return tile[ch][oc]; });
  }
  if (wT && !frag_transpose) {
#pragma unroll
    for (int p = 0; p < kPasses; ++p) {
      const int c = c0 + row + kRows * p, k = k0 + col, at = row + kRows * p;
      if (c < C && k < K) store4(wT + ((size_t)c * RS + tap) * K + k, tile[col][at], tile[col + 1][at], tile[col + 2][at], tile[col + 3][at]);
    }
  }
}

template <int N, int TS = 64>
int prepare_launch(const std::vector<FilterPrep> &items, int dt, hipStream_t st, int src_dt) {
  size_t i = 0;
  while (i < items.size()) {
    PrepTable<N> t{};
    int wg = 0;
    double bytes = 0;
    while (i < items.size() && t.nseg < N) {
      const FilterPrep &f = items[i++];
      if ((f.g.K & 3) || (f.g.C & 3)) return set_error(RESIST_ESHAPE, "filter %dx%d: channel counts must be multiples of 4", f.g.K, f.g.C);
      if (!f.w_lp && !f.wT) continue;
      const int n = t.nseg++;
      t.w[n] = f.w; t.wlp[n] = f.w_lp; t.wT[n] = f.wT;
      t.K[n] = f.g.K; t.RS[n] = f.g.R * f.g.S; t.C[n] = f.g.C;
      t.scale[n] = f.scale;
      if (f.lp_fragments) t.frag_copy |= 1ull << n;
      if (f.wT_fragments) t.frag_transpose |= 1ull << n;
      t.first_wg[n] = wg;
      wg += ((f.g.C + 63) / 64) * ((f.g.K + 63) / 64) * f.g.R * f.g.S;
      bytes += (double)esize(src_dt) * f.g.K * f.g.R * f.g.S * f.g.C + (f.w_lp ? filter_bytes(f.g, dt, f.lp_fragments, false) : 0) + (f.wT ? filter_bytes(f.g, dt, f.wT_fragments, true) : 0);
    }
    t.first_wg[t.nseg] = wg;
    if (wg == 0) continue;
    prof::Scope ps("prepare_filters", 0, bytes, st);
    const dim3 grid = N == 1 ? dim3((t.C[0] + TS - 1) / TS, (t.K[0] + TS - 1) / TS, t.RS[0]) : dim3(wg);
    if (src_dt == DT_BF16) hipLaunchKernelGGL((prepare_filters_kernel<__bf16, __bf16, N, TS>), grid, dim3(256), 0, st, t);
    else if (dt == DT_BF16) hipLaunchKernelGGL((prepare_filters_kernel<float, __bf16, N, TS>), grid, dim3(256), 0, st, t);
    else hipLaunchKernelGGL((prepare_filters_kernel<float, float, N, TS>), grid, dim3(256), 0, st, t);
    RESIST_CHECK_LAUNCH("prepare_filters");
  }
  return RESIST_OK;
}
}  // namespace

int prepare_filters(const std::vector<FilterPrep> &items, int dt, hipStream_t st, int src_dt) {
  if (src_dt == DT_BF16 && dt != DT_BF16) return set_error(RESIST_EINVAL, "prepare_filters: bf16 source needs a bf16 target");
  if (items.size() > 1) return prepare_launch<kPrepSegs>(items, dt, st, src_dt);
  const bool fragments = !items.empty() && ((items[0].w_lp && items[0].lp_fragments) || (items[0].wT && items[0].wT_fragments));
  return fragments ? prepare_launch<1>(items, dt, st, src_dt) : prepare_launch<1, 32>(items, dt, st, src_dt);
}

// ---- wgrad --------------------------------------------------------------------------------------
namespace {

constexpr int kWBK = 32;  // reduction rows staged per step

struct WgradArgs {
  const void *dy;   // [M][K]
  const void *x;    // [N][H][W][C]
  float *out;       // [splits][K][R][S][C]
  int N, H, W, C, K, R, S, stride, pad, P, Q;
  int M;            // N*P*Q
  int rows_per_split;
  int tiles_k, tiles_c;
  FastDiv div_pq, div_q;
};

// Weight gradient: rows of the GEMM are output channels, columns are input channels of one filter
// tap, the reduction runs over output pixels m (split across workgroups).  Both operand tiles arrive
// "reduction-major" ([m][channel]) straight from the NHWC tensors.  Same pipeline as the forward
// kernel: straight-line loop body, bounds-checked buffer loads, LDS refill in the middle of the
// MFMAs, fragments fetched one k-step ahead.  This is the fp32 kernel: the matrix instruction takes
// one reduction index per lane, so fragments are single LDS words and no transpose is needed.
template <int BM, int BN, int WGM, int WGN>
__global__ __launch_bounds__(kThreads) void wgrad_kernel(WgradArgs a) {
  constexpr int VEC = 4;
  constexpr int ES = 4;
  constexpr int WTM = BM / WGM, WTN = BN / WGN;
  constexpr int TM = WTM / 32, TN = WTN / 32;
  constexpr int LDA = BM + 32, LDB = BN + 32;     // rows kk and kk+1 land on different bank halves
  constexpr int TPRA = BM / VEC, TPRB = BN / VEC; // threads per 32-row-chunk row
  constexpr int RPA = kThreads / TPRA, RPB = kThreads / TPRB;  // rows per pass
  constexpr int PA = (kWBK + RPA - 1) / RPA, PB = (kWBK + RPB - 1) / RPB;
  constexpr int NK = kWBK / 2;
  __shared__ float As[2][kWBK][LDA];
  __shared__ float Bs[2][kWBK][LDB];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WGN, wn = wave % WGN;
  // order: tile fastest, then filter tap, then reduction split; every XCD gets one contiguous range
  // of that order, i.e. a range of reduction rows, so each L2 fetches only its share of dy and x
  // (with the hardware's round-robin order every XCD read both tensors in full: 8x the traffic, same speed)
  int bid = xcd_contiguous(blockIdx.x, gridDim.x);
  const int tile = bid % (a.tiles_k * a.tiles_c);
  bid /= a.tiles_k * a.tiles_c;
  const int tap = bid % (a.R * a.S), split = bid / (a.R * a.S);
  const int tk = tile / a.tiles_c, tc = tile % a.tiles_c;
  const int r = tap / a.S, s = tap - r * a.S;
  const int k0 = tk * BM, c0 = tc * BN;
  const int mbeg = split * a.rows_per_split;
  const int mend = min(a.M, mbeg + a.rows_per_split);
  const int nchunks = (mend - mbeg + kWBK - 1) / kWBK;

  const int arow = tid / TPRA, acol = (tid % TPRA) * VEC;
  const int brow = tid / TPRB, bcol = (tid % TPRB) * VEC;
  const unsigned acolb = (k0 + acol) < a.K ? (unsigned)(k0 + acol) * ES : kOOB;
  const unsigned bcolb = (c0 + bcol) < a.C ? (unsigned)(c0 + bcol) * ES : kOOB;
  const __amdgpu_buffer_rsrc_t rdy = make_rsrc(a.dy, (unsigned)a.M * a.K * ES);
  const __amdgpu_buffer_rsrc_t rx = make_rsrc(a.x, (unsigned)a.N * a.H * a.W * a.C * ES);

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  f32x4 ra[PA], rb[PB];
  int mc = mbeg;   // first reduction row of the chunk being requested
  // register `part` (0..PA-1: rows of dy, PA..PA+PB-1: rows of x) of the chunk starting at row mc
  auto request = [&](int part) {
    if (part < PA) {
      const int row = part * RPA + arow;
      const int m = mc + row;
      ra[part] = buffer_load_16B(rdy, (m < mend && row < kWBK) ? (unsigned)m * (unsigned)a.K * ES + acolb : kOOB);
    } else {
      const int i = part - PA;
      const int row = i * RPB + brow;
      const int m = mc + row;
      const int n = fdiv(m, a.div_pq);
      const int rem = m - n * (a.P * a.Q);
      const int p = fdiv(rem, a.div_q), q = rem - p * a.Q;
      const int ih = p * a.stride + r - a.pad, iw = q * a.stride + s - a.pad;
      const bool ok = m < mend && row < kWBK && (unsigned)ih < (unsigned)a.H && (unsigned)iw < (unsigned)a.W;
      rb[i] = buffer_load_16B(rx, ok ? (unsigned)((n * a.H + ih) * a.W + iw) * (unsigned)a.C * ES + bcolb : kOOB);
    }
  };
  auto store_part = [&](int stage, int part) {
    if (part < PA) {
      if (part * RPA + arow < kWBK) *reinterpret_cast<f32x4 *>(&As[stage][part * RPA + arow][acol]) = ra[part];
    } else {
      const int i = part - PA;
      if (i * RPB + brow < kWBK) *reinterpret_cast<f32x4 *>(&Bs[stage][i * RPB + brow][bcol]) = rb[i];
    }
  };
  auto load_global = [&]() {
#pragma unroll
    for (int p = 0; p < PA + PB; ++p) request(p);
    mc += kWBK;
  };
  auto store_lds = [&](int stage) {
#pragma unroll
    for (int p = 0; p < PA + PB; ++p) store_part(stage, p);
  };

  // same pipeline as the forward kernel: fragments one k-step ahead (also across chunks), refill of
  // the other stage spread over k-steps 0 .. NK-2, one barrier per chunk at the start of the last k-step
  static_assert(NK % 2 == 0, "fragment double buffer parity");
  const int lr = lane & 31, lh = lane >> 5;
  float fa[2][TM], fb[2][TN];
  auto load_frags = [&](int buf, int stage, int ks) {
#pragma unroll
    for (int i = 0; i < TM; ++i) fa[buf][i] = As[stage][ks * 2 + lh][wm * WTM + i * 32 + lr];
#pragma unroll
    for (int j = 0; j < TN; ++j) fb[buf][j] = Bs[stage][ks * 2 + lh][wn * WTN + j * 32 + lr];
  };
  auto lds_barrier = [&]() {
    __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
  };
  load_global();
  store_lds(0);
  load_global();
  lds_barrier();
  load_frags(0, 0, 0);
  __builtin_amdgcn_sched_barrier(0);
  for (int it = 0; it < nchunks; ++it) {
    const int stage = it & 1;
#pragma unroll
    for (int ks = 0; ks < NK; ++ks) {
      if (ks + 1 < NK) {
        load_frags((ks + 1) & 1, stage, ks + 1);
      } else {
        lds_barrier();
        load_frags(0, stage ^ 1, 0);   // rows past mend were loaded as zeros
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int p = 0; p < PA + PB; ++p)
        if ((p * (NK - 1)) / (PA + PB) == ks) {   // refill spread evenly over k-steps 0 .. NK-2
          store_part(stage ^ 1, p);
          request(p);
        }
      if (ks == NK - 2) mc += kWBK;
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[ks & 1][i], fb[ks & 1][j], acc[i][j], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  float *out = a.out + (size_t)split * a.K * a.R * a.S * a.C;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int c = c0 + wn * WTN + j * 32 + lr;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int k = k0 + wm * WTM + i * 32 + (e >> 2) * 8 + lh * 4 + (e & 3);
        if (k < a.K && c < a.C) out[((size_t)k * a.R * a.S + tap) * a.C + c] = acc[i][j][e];
      }
    }
}

// Weight gradient with bf16 operands on v_mfma_f32_32x32x16_bf16.  The matrix instruction wants 8
// consecutive values of the reduction index (output pixels m) per lane, while both operands arrive
// from memory with the channel index contiguous ([m][channel]); the tiles are therefore stored in LDS
// as they arrive and read back through the LDS transpose read, two 4-deep reads per fragment.
// WBK: pixels staged per chunk (a multiple of 32); otherwise the same pipeline as the fp32 kernel.
template <int BM, int BN, int WBK>
__global__ __launch_bounds__(kThreads) void wgrad_bf16_kernel(WgradArgs a) {
  constexpr int WGM = 2, WGN = 2;
  constexpr int WTM = BM / WGM, WTN = BN / WGN;
  constexpr int TM = WTM / 32, TN = WTN / 32;
  constexpr int LDA = BM + 32, LDB = BN + 32;     // row pitch = tile width + 64 bytes: 4 consecutive rows fall on disjoint banks
  constexpr int TPRA = BM / 8, TPRB = BN / 8;     // threads per tile row (16 bytes each)
  constexpr int RPA = kThreads / TPRA, RPB = kThreads / TPRB;
  constexpr int PA = WBK / RPA, PB = WBK / RPB;
  constexpr int NK = WBK / 16;
  static_assert(WBK % RPA == 0 && WBK % RPB == 0 && NK % 2 == 0 && TM >= 1 && TN >= 1, "tile shape");
  __shared__ __bf16 As[2][WBK][LDA];
  __shared__ __bf16 Bs[2][WBK][LDB];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WGN, wn = wave % WGN;
  // every XCD gets a contiguous range of (tile, tap, split) ids, so the workgroups that read the same
  // pixels (all tiles and taps of one split) share an L2: this kernel is bound by memory traffic
  int bid = xcd_contiguous(blockIdx.x, gridDim.x);
  const int tile = bid % (a.tiles_k * a.tiles_c);
  bid /= a.tiles_k * a.tiles_c;
  const int tap = bid % (a.R * a.S), split = bid / (a.R * a.S);
  const int tk = tile / a.tiles_c, tc = tile % a.tiles_c;
  const int r = tap / a.S, s = tap - r * a.S;
  const int k0 = tk * BM, c0 = tc * BN;
  const int mbeg = split * a.rows_per_split;
  const int mend = min(a.M, mbeg + a.rows_per_split);
  const int nchunks = (mend - mbeg + WBK - 1) / WBK;

  const int arow = tid / TPRA, acol = (tid % TPRA) * 8;
  const int brow = tid / TPRB, bcol = (tid % TPRB) * 8;
  const unsigned acolb = (k0 + acol) < a.K ? (unsigned)(k0 + acol) * 2u : kOOB;
  const unsigned bcolb = (c0 + bcol) < a.C ? (unsigned)(c0 + bcol) * 2u : kOOB;
  const __amdgpu_buffer_rsrc_t rdy = make_rsrc(a.dy, (unsigned)a.M * a.K * 2u);
  const __amdgpu_buffer_rsrc_t rx = make_rsrc(a.x, (unsigned)a.N * a.H * a.W * a.C * 2u);

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  f32x4 ra[PA], rb[PB];
  int mc = mbeg;   // first reduction row of the chunk being requested
  auto request = [&](int part) {
    if (part < PA) {
      const int m = mc + part * RPA + arow;
      ra[part] = buffer_load_16B(rdy, m < mend ? (unsigned)m * (unsigned)a.K * 2u + acolb : kOOB);
    } else {
      const int i = part - PA;
      const int m = mc + i * RPB + brow;
      const int n = fdiv(m, a.div_pq);
      const int rem = m - n * (a.P * a.Q);
      const int p = fdiv(rem, a.div_q), q = rem - p * a.Q;
      const int ih = p * a.stride + r - a.pad, iw = q * a.stride + s - a.pad;
      const bool ok = m < mend && (unsigned)ih < (unsigned)a.H && (unsigned)iw < (unsigned)a.W;
      rb[i] = buffer_load_16B(rx, ok ? (unsigned)((n * a.H + ih) * a.W + iw) * (unsigned)a.C * 2u + bcolb : kOOB);
    }
  };
  auto store_part = [&](int stage, int part) {
    if (part < PA) *reinterpret_cast<f32x4 *>(&As[stage][part * RPA + arow][acol]) = ra[part];
    else *reinterpret_cast<f32x4 *>(&Bs[stage][(part - PA) * RPB + brow][bcol]) = rb[part - PA];
  };
  auto load_global = [&]() {
#pragma unroll
    for (int p = 0; p < PA + PB; ++p) request(p);
    mc += WBK;
  };
  auto store_lds = [&](int stage) {
#pragma unroll
    for (int p = 0; p < PA + PB; ++p) store_part(stage, p);
  };

  // fragment addressing of the transpose read: lane l supplies row 8*(l/32) + (l%16)/4 of a 16-row
  // k-step and columns 16*((l/16)%2) + 4*(l%4) .. +3 of a 32-column tile; it receives column l%32,
  // rows 8*(l/32) .. +3 (and +4 .. +7 from the second read)
  const int frow = (lane >> 5) * 8 + ((lane & 15) >> 2);
  const int fcol = ((lane >> 4) & 1) * 16 + (lane & 3) * 4;
  bf16x8 fa[2][TM], fb[2][TN];
  auto load_frags = [&](int buf, int stage, int ks) {
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      fa[buf][i] = lds_read_tr_pair(&As[stage][ks * 16 + frow][wm * WTM + i * 32 + fcol],
                                    &As[stage][ks * 16 + frow + 4][wm * WTM + i * 32 + fcol]);
    }
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      fb[buf][j] = lds_read_tr_pair(&Bs[stage][ks * 16 + frow][wn * WTN + j * 32 + fcol],
                                    &Bs[stage][ks * 16 + frow + 4][wn * WTN + j * 32 + fcol]);
    }
  };
  auto lds_barrier = [&]() {
    __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
  };
  load_global();
  store_lds(0);
  load_global();
  lds_barrier();
  load_frags(0, 0, 0);
  __builtin_amdgcn_sched_barrier(0);
  for (int it = 0; it < nchunks; ++it) {
    const int stage = it & 1;
#pragma unroll
    for (int ks = 0; ks < NK; ++ks) {
      if (ks + 1 < NK) {
        load_frags((ks + 1) & 1, stage, ks + 1);
      } else {
        lds_barrier();
        load_frags(0, stage ^ 1, 0);   // rows past mend were loaded as zeros
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int p = 0; p < PA + PB; ++p)
        if ((p * (NK - 1)) / (PA + PB) == ks) {   // refill spread evenly over k-steps 0 .. NK-2
          store_part(stage ^ 1, p);
          request(p);
        }
      if (ks == NK - 2) mc += WBK;
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[ks & 1][i], fb[ks & 1][j], acc[i][j], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  const int lr = lane & 31, lh = lane >> 5;
  float *out = a.out + (size_t)split * a.K * a.R * a.S * a.C;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int c = c0 + wn * WTN + j * 32 + lr;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int k = k0 + wm * WTM + i * 32 + (e >> 2) * 8 + lh * 4 + (e & 3);
        if (k < a.K && c < a.C) out[((size_t)k * a.R * a.S + tap) * a.C + c] = acc[i][j][e];
      }
    }
}

// Sum of the split partial results, in a fixed order (bit-stable from run to run): thread (x, g)
// adds splits g, g+G, g+2G, ... of output vector x in ascending order, then the G partial sums are
// added in ascending g.  G threads share one output vector so that many loads are in flight even
// when the output is small and the number of splits large.
template <int G>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const float *__restrict__ part, float *__restrict__ out,
                                                            long long n4, int splits) {
  constexpr int X = 256 / G;
  __shared__ f32x4 red[G][X];
  const int x = threadIdx.x % X, g = threadIdx.x / X;
  const long long i = (long long)blockIdx.x * X + x;
  const f32x4 *p = reinterpret_cast<const f32x4 *>(part);
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  if (i < n4)
    for (int z = g; z < splits; z += G) acc += p[i + (long long)z * n4];
  if (G > 1) {
    red[g][x] = acc;
    __syncthreads();
    if (g == 0) {
#pragma unroll
      for (int h = 1; h < G; ++h) acc += red[h][x];
    }
  }
  if (g == 0 && i < n4) reinterpret_cast<f32x4 *>(out)[i] = acc;
}

constexpr size_t kStaticScratchBytes = (size_t)32 << 20;   // library-owned partial sums (see conv_wgrad_static)

struct WgradPlan { int bm, bn, splits, rows_per_split; bool taps9 = false, taps3 = false; };

// Nine-tap kernel (wgrad3.hip): 64 x 64 channels of all taps per workgroup, one workgroup per CU, in a step as alone.  (128
// workgroups beside the data gradients of a step, with half the partial sums, were 3 % of a step faster, 4427 -> 4295 us for the CIFAR-shaped
// sub-ResNet, batch 128, but an accumulator then runs over twice the rows: error against float64 1.14e-7 -> 1.41e-7 at
// 256 ch 8x8, 1.53e-7 -> 1.90e-7 at 128 ch 28x28.  128 workgroups of two such ranges each, one after the other: 4452 us.)  Its time is that of
// the rounds of 256 workgroups, 0.05 us per row and 128 rows' worth for its start and end, 0.06 us per partial tile
// written and read back, 4 us for the launch that adds them; the number of splits is the one with the least, among those whose partial sums stay below
// max_floats.
WgradPlan plan_wgrad3(const ConvGeom &g, long long max_floats) {
  WgradPlan p;
  p.bm = p.bn = 64;
  p.taps9 = true;
  const long long tiles = (long long)((g.K + 63) / 64) * ((g.C + 63) / 64), M = (long long)g.N * g.P * g.Q;
  const long long slice = (long long)g.K * 9 * g.C;
  long long best = -1;
  for (long long s = 1; s <= 256 && (s == 1 || (s - 1) * 64 < M); ++s) {
    if (s > 1 && s * slice > max_floats) break;
    const long long rows = ((M + s - 1) / s + kWBK - 1) / kWBK * kWBK;
    const long long used = (M + rows - 1) / rows;
    const long long cost = (tiles * used + 255) / 256 * (rows + 128) * 5 + (used > 1 ? tiles * used * 6 + 400 : 0);
    if (best < 0 || cost < best) { best = cost; p.splits = (int)used; p.rows_per_split = (int)rows; }
  }
  return p;
}

// One filter row per workgroup (wgrad3_row_bf16_kernel).  In a step, as many splits as give 384
// workgroups, which leaves compute units room for the data gradients (CIFAR-shaped model, batch 128: 256 workgroups 5.70 ms, 384 5.65, 512
// 5.72; 256 are no slower since the output gradients take turns in six buffers, but add up longer, 1.04e-7 -> 1.27e-7 against
// float64 at 256 ch 8x8).  Alone, one workgroup for every compute unit, or two where the reduction is long enough to pay for the partial sums,
// from 3 * 2^28 padded products a tap: us, up to 256 | 384 | 512 workgroups (one tap a workgroup), 256 ch 8x8, batch 128 29.6 |
// 30.9 | 31.0 (29.7), 16x16 128 ch, batch 77 23.7 | 27.2 | 26.7 (24.2), 14x14 256 ch, batch 64 36.3 | 39.0 | 33.7 (38.7), batch 256
// 104 | 104 | 90 (134).  A second split of 192 or more tiles costs as much in partial sums as it saves (512 -> 512 channels at
// 7x7, batch 64: 36 us in one, 32 + 5 in two; batch 8: 12 and 17 + 6).
WgradPlan plan_wgrad_rows(const ConvGeom &g, bool step) {
  WgradPlan p;
  p.bm = p.bn = 64;
  p.taps3 = true;
  const long long tiles = (long long)((g.K + 63) / 64) * ((g.C + 63) / 64) * 3, M = (long long)g.N * g.P * g.Q;
  const long long wgs = step ? 384 : M * tiles >= 9LL << 16 ? 512 : 256;
  long long splits = std::min(wgs / tiles, (M + 255) / 256);
  if (tiles >= 192 || (step && splits <= 2) || splits < 1) splits = 1;
  const long long rows = ((M + splits - 1) / splits + 63) / 64 * 64;
  p.rows_per_split = (int)rows;
  p.splits = (int)((M + rows - 1) / rows);
  return p;
}

WgradPlan plan_wgrad(const ConvGeom &g) {
  WgradPlan p;
  p.bm = p.bn = wgrad_tile(g);
  const long long tiles = (long long)((g.K + p.bm - 1) / p.bm) * ((g.C + p.bn - 1) / p.bn) * g.R * g.S;
  const long long M = (long long)g.N * g.P * g.Q;
  long long splits = 768 / tiles;   // at most three workgroups per CU: all resident at once (measured best)
  const long long max_splits = (M + 255) / 256;  // at least 256 reduction rows per split
  if (splits > max_splits) splits = max_splits;
  if (splits < 1) splits = 1;
  if (splits > 256) splits = 256;
  long long rps = (M + splits - 1) / splits;
  rps = (rps + kWBK - 1) / kWBK * kWBK;
  p.rows_per_split = (int)rps;
  p.splits = (int)((M + rps - 1) / rps);
  return p;
}

}  // namespace

namespace {
int64_t plan_floats(const WgradPlan &p, const ConvGeom &g) { return p.splits > 1 ? (int64_t)p.splits * g.K * g.R * g.S * g.C : 0; }

int run_wgrad(const WgradPlan &p, const ConvGeom &g, int dt, const void *dy, const void *x, float *dw, float *partial, hipStream_t st) {
  if (p.splits > 1 && !partial) return set_error(RESIST_EWORKSPACE, "wgrad needs split scratch");
  if (p.taps9) {
    {
      const double M = (double)g.N * g.P * g.Q;
      prof::Scope ps("wgrad3_f32", 2.0 * M * g.K * g.C * 9, 4.0 * (M * (g.K + g.C) + 9.0 * g.K * g.C), st);
      RESIST_TRY(wgrad3_launch(g, static_cast<const float *>(dy), static_cast<const float *>(x), p.splits > 1 ? partial : dw, p.splits,
                               p.rows_per_split, st));
    }
    return p.splits > 1 ? splitk_reduce(partial, dw, (long long)g.K * 9 * g.C / 4, p.splits, st) : RESIST_OK;
  }
  if (p.taps3) {
    {
      const double M = (double)g.N * g.P * g.Q;
      prof::Scope ps("wgrad3_row_bf16", 2.0 * M * g.K * g.C * 9, 2.0 * M * (g.K + g.C) + 36.0 * g.K * g.C, st);
      RESIST_TRY(wgrad3_row_launch(g, dy, x, p.splits > 1 ? partial : dw, p.splits, p.rows_per_split, st));
    }
    return p.splits > 1 ? splitk_reduce(partial, dw, (long long)g.K * 9 * g.C / 4, p.splits, st) : RESIST_OK;
  }
  WgradArgs a{};
  a.dy = dy; a.x = x; a.out = p.splits > 1 ? partial : dw;
  a.N = g.N; a.H = g.H; a.W = g.W; a.C = g.C; a.K = g.K; a.R = g.R; a.S = g.S;
  a.stride = g.stride; a.pad = g.pad; a.P = g.P; a.Q = g.Q;
  a.M = g.N * g.P * g.Q;
  a.rows_per_split = p.rows_per_split;
  a.tiles_k = (g.K + p.bm - 1) / p.bm;
  a.tiles_c = (g.C + p.bn - 1) / p.bn;
  a.div_pq = make_fastdiv((unsigned)(g.P * g.Q));
  a.div_q = make_fastdiv((unsigned)g.Q);
  dim3 grid((unsigned)(a.tiles_k * a.tiles_c * g.R * g.S * p.splits));
  {
    const double flops = 2.0 * a.M * g.K * g.C * g.R * g.S;
    const double bytes = esize(dt) * ((double)a.M * g.K + (double)g.N * g.H * g.W * g.C) + 4.0 * g.K * g.R * g.S * g.C;
    const char *label = dt == DT_BF16 ? (p.bm == 128 ? "wgrad_bf16_128x128" : "wgrad_bf16_64x64")
                                      : (p.bm == 128 ? "wgrad_f32_128x128" : "wgrad_f32_64x64");
    prof::Scope ps(label, flops, bytes, st);
    if (dt == DT_BF16) {
      if (p.bm == 128) hipLaunchKernelGGL((wgrad_bf16_kernel<128, 128, 32>), grid, dim3(kThreads), 0, st, a);
      else hipLaunchKernelGGL((wgrad_bf16_kernel<64, 64, 64>), grid, dim3(kThreads), 0, st, a);
    } else {
      if (p.bm == 128) hipLaunchKernelGGL((wgrad_kernel<128, 128, 2, 2>), grid, dim3(kThreads), 0, st, a);
      else hipLaunchKernelGGL((wgrad_kernel<64, 64, 2, 2>), grid, dim3(kThreads), 0, st, a);
    }
  }
  RESIST_CHECK_LAUNCH("wgrad");
  if (p.splits > 1) return splitk_reduce(partial, dw, (long long)g.K * g.R * g.S * g.C / 4, p.splits, st);
  return RESIST_OK;
}

}  // namespace

int wgrad_tile(const ConvGeom &g) {
  return g.K >= 128 && g.C >= 128 && (long long)g.K * g.C * g.R * g.S >= 128LL * 128 * 9 * 16 ? 128 : 64;
}

// A layer whose one-tap plan fits the static scratch has a nine-tap plan that fits it too: conv_wgrad_static takes the
// same layers, and gives the same bits as conv_wgrad, whichever kernel runs.
static WgradPlan plan_for(const ConvGeom &g, int dt, bool step = false) {
  const WgradPlan p = plan_wgrad(g);
  if (dt == DT_BF16 && wgrad3_row_takes(g)) return plan_wgrad_rows(g, step);   // at most 25 MB of partial sums
  if (dt != DT_F32 || !wgrad3_takes(g)) return p;
  return plan_wgrad3(g, plan_floats(p, g) * 4 <= (int64_t)kStaticScratchBytes ? (long long)(kStaticScratchBytes / 4) : INT64_MAX);
}

int64_t wgrad_scratch_floats(const ConvGeom &g, int dt, bool step) { return plan_floats(plan_for(g, dt, step), g); }

int64_t wgrad_reserve_floats(const ConvGeom &g, int dt) { return std::max(wgrad_scratch_floats(g, dt), plan_floats(plan_wgrad(g), g)); }

int conv_wgrad(const ConvGeom &g, int dt, const void *dy, const void *x, float *dw, float *partial, hipStream_t st, bool step) {
  RESIST_TRY(check_geom(g, dt));
  return run_wgrad(plan_for(g, dt, step), g, dt, dy, x, dw, partial, st);
}

int splitk_reduce(const float *partial, float *out, long long n4, int splits, hipStream_t st) {
  prof::Scope ps("splitk_reduce", 0, 16.0 * n4 * (splits + 1), st);
  // enough threads per output vector that the launch has at least ~64k loads in flight
  if (n4 * 4 >= 65536 || splits < 8)
    hipLaunchKernelGGL(splitk_reduce_kernel<4>, dim3((unsigned)((n4 + 63) / 64)), dim3(256), 0, st, partial, out, n4, splits);
  else
    hipLaunchKernelGGL(splitk_reduce_kernel<16>, dim3((unsigned)((n4 + 15) / 16)), dim3(256), 0, st, partial, out, n4, splits);
  RESIST_CHECK_LAUNCH("splitk_reduce");
  return RESIST_OK;
}

// ---- weight gradient with its split partial sums in library-owned static device memory ------------
// For callers that cannot allocate (HIP graph capture, serving loops): the split-reduction scratch of
// conv_wgrad lives in a file-scope device array instead of a caller-provided workspace.  Host code
// never uses the array's name as an address: its device address is looked up once per device.
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {
constexpr int kScratchDevices = 16;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kScratchDevices] = {};

// device address of `scratch` on the current device (each GPU holds its own copy at its own address)
int static_scratch(void **out) {
  int dev = 0;
  RESIST_CHECK_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kScratchDevices) return set_error(RESIST_EUNSUPPORTED, "device %d: at most %d devices", dev, kScratchDevices);
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void *p = nullptr;
    RESIST_CHECK_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p) return set_error(RESIST_EHIP, "hipGetSymbolAddress returned NULL");
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return RESIST_OK;
}
}  // namespace

int64_t wgrad_static_scratch_bytes() { return (int64_t)kStaticScratchBytes; }

int conv_wgrad_static(const ConvGeom &g, int dt, const void *dy, const void *x, float *dw, hipStream_t st) {
  RESIST_TRY(check_geom(g, dt));
  const int64_t need = wgrad_reserve_floats(g, dt) * 4;
  if (need > (int64_t)kStaticScratchBytes)
    return set_error(RESIST_EWORKSPACE, "split partial sums: %lld bytes reserved for this shape, the static scratch holds %lld",
                     (long long)need, (long long)kStaticScratchBytes);
  void *ptr = nullptr;
  RESIST_TRY(static_scratch(&ptr));
  // every split writes its whole [K][R][S][C] slice before the reduction reads it: nothing to clear
  return conv_wgrad(g, dt, dy, x, dw, need > 0 ? static_cast<float *>(ptr) : nullptr, st);
}

}  // namespace resist
