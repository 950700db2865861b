// Device-side parts shared by the convolution kernels (conv.hip, conv3.hip): element traits, launch arguments,
// tile order, bounds-checked loads and the epilogue that takes a tile from the accumulators to memory.
#pragma once
#include <type_traits>

#include "elem.h"
#include "internal.h"

namespace resist {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// division by a runtime constant: q = (n * mul) >> sh, exact for 0 <= n < 2^31
struct FastDiv { unsigned mul; int sh; };
inline FastDiv make_fastdiv(unsigned d) {
  int L = 0;
  while ((1ull << L) < d) ++L;
  FastDiv f;
  f.sh = 31 + L;
  f.mul = (unsigned)((1ull << f.sh) / d + 1);
  return f;
}
__device__ inline int fdiv(int n, FastDiv f) { return (int)(((unsigned long long)(unsigned)n * f.mul) >> f.sh); }

struct IgemmArgs {
  const void *in;      // [N][IH][IW][IC]
  const void *wt;      // [OC][R][S][IC]
  void *out;           // [N][OH][OW][OC]
  const void *addend;  // optional, indexed like out
  const void *relu_mask;   // optional, indexed like out: out is zeroed where this is not positive (after the addend)
  float *stats;        // optional [3][tiles_m][OC]: per row tile and column a shift k, sum(out - k), sum((out - k)^2)
  // optional (data gradient, cls == 1): first pass of the backward of the BN whose output this
  // convolution read.  out is that BN's output gradient g; with its input bn_y (indexed like out) and
  // xhat = (bn_y - mean) * invstd the kernel leaves, per row tile and column, sum(gm) and sum(gm * xhat) in
  // bn_sums [2][tiles_m][OC], where gm = g, or g where scale * bn_y + shift > 0 and 0 elsewhere (bn_self)
  const void *bn_y;
  const float *bn_mean, *bn_invstd, *bn_scale, *bn_shift;
  float *bn_sums;
  int bn_self;
  int N, IH, IW, IC;
  int OH, OW, OC;
  int R, S, stride, pad;
  int cls;              // 1, or 2 when output pixels are split into 2x2 parity classes
  int OHc, OWc;         // OH/cls, OW/cls
  int Mrows;            // N*OHc*OWc: GEMM rows per class
  int tiles_m, tiles_n;
  FastDiv div_plane, div_w, div_tn, div_tm;   // by OHc*OWc, OWc, tiles_n, tiles_m: a tile's prologue is a chain of divisions
};

// of a streamed 1x1 convolution: pixels per workgroup and how many such ranges there are
struct Conv1Args : IgemmArgs { int rows, parts; };

// A-gather modes
constexpr int kFwd = 0;  // source pixel = out*stride + tap - pad
constexpr int kBwd = 1;  // source pixel = (out + pad - tap) / stride
// as kFwd, and the affine map, shortcut and ReLU of the BN behind it applied to the tile before it is stored: at test
// time the map is known beforehand, so a separate pass (read y, read the shortcut, write a: 5 us a layer and as much again
// for the launch that made its map) buys nothing.  CIFAR-shaped model, batch 128, fp32: 6.04 -> 5.56 ms; batch 33, bf16:
// 1.48 -> 1.05; one ImageNet-shaped image, bf16: 0.83 -> 0.55; bit for bit the same logits.
constexpr int kEval = 2;
// Its arguments.  The other kernels are launched without them: a longer argument block puts what the launch appends to it
// (grid size) in another cache line, 0.1 us of every launch.
struct EvalArgs : IgemmArgs {
  // out (if not NULL) is stored as above, and v, the value as stored there, goes on to
  //   act = max(act_scale*v + act_shift [+ res_scale*act_res + res_shift], 0)    (NULL res_scale: + act_res)
  void *act;
  const float *act_scale, *act_shift;
  const void *act_res;
  const float *res_scale, *res_shift;
};
template <int MODE> using ArgsOf = std::conditional_t<MODE == kEval, EvalArgs, IgemmArgs>;
// of a convolution on a prepared filter
template <int MODE> struct Conv3Args : ArgsOf<MODE> {
  const void *frag;
  const unsigned *flags;   // behind the fragments: which hold operands that three parts do not
  float wscale;
  int cchunks, m_fast, share, ahead;
};

namespace {

// Element traits: a 16-byte vector holds VEC elements; one pair of 16-byte fragments (A, B) feeds
// the matrix core with 2*VEC values of the GEMM-K axis (lane group l/32 owns VEC consecutive ones).
template <typename T> struct Elem;
template <> struct Elem<float> {
  static constexpr int VEC = 4;
  __device__ static inline void mma(f32x16 &acc, const f32x4 &a, const f32x4 &b) {
#pragma unroll
    for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[e], b[e], acc, 0, 0, 0);
  }
  __device__ static inline float from_f32(float v) { return v; }
  __device__ static inline float to_f32(float v) { return v; }
};
template <> struct Elem<__bf16> {
  static constexpr int VEC = 8;
  __device__ static inline void mma(f32x16 &acc, const f32x4 &a, const f32x4 &b) {
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
  }
  __device__ static inline __bf16 from_f32(float v) { return (__bf16)v; }   // round to nearest even
  __device__ static inline float to_f32(__bf16 v) { return (float)v; }
};

// The leading bf16 part of four fp32 values (nearest even), packed; v keeps what it leaves, exactly.  Three calls take a
// value apart: 8 + 8 + 8 significant bits.  (An infinity, or a value that rounds to one, leaves a NaN behind.)
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
__device__ inline u32x2 split_part(f32x4 &v) {
  const unsigned a = __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2{v[0], v[1]}), bf16x2));
  const unsigned b = __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2{v[2], v[3]}), bf16x2));
  v -= f32x4{bf16_lo(a), bf16_hi(a), bf16_lo(b), bf16_hi(b)};
  return u32x2{a, b};
}
// Between the second call and the third: adds to `missed` the lanes whose parts may not hold all of a value.  The last bit of
// bf16's smallest numbers is 2^-133, so below 2^-110 the parts of a value run out of bits; what two parts leave of such a
// value is a subnormal float (and of values from 2^-103 up it never is).  It costs the forward kernel 2 % and the data
// gradient 1 (14x14, 256 ch, batch 64: 88.8 -> 90.9 us, 96.4 -> 97.9; the largest or the smallest magnitude of what is staged
// instead: the same or more).
__device__ inline void split_check(const f32x4 &v, unsigned long long &missed) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {   // one instruction into a scalar mask; the builtin of it goes through a vector register
    unsigned long long lanes;
    asm("v_cmp_class_f32 %0, %1, %2" : "=s"(lanes) : "v"(v[e]), "s"(0x90));   // subnormal of either sign
    missed |= lanes;
  }
}

// LDS transpose read (ds_read_b64_tr_b16).  Within each block of 16 lanes, lane s supplies the
// address of 4 consecutive 16-bit values; lane j receives, as element e, the value number j%4 of
// the four that lane 4*e + j/4 pointed at.  When lane s points at row s/4, columns 4*(s%4)..+3 of a
// row-major tile, lane j therefore ends up with rows 0..3 of column j: a 4x16 -> 16x4 transpose.
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
__device__ inline s16x4 lds_read_tr(const void *p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(p));
}
// two of them: eight consecutive values of the reduction index for the matrix instruction
__device__ inline bf16x8 lds_read_tr_pair(const void *first, const void *second) {
  const s16x4 lo = lds_read_tr(first), hi = lds_read_tr(second);
  return __builtin_bit_cast(bf16x8, (s16x8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]}));
}

// Workgroups are handed to the 8 XCDs round-robin by their linear id, and each XCD has its own L2.
// This maps the hardware id to a logical tile index such that every XCD works on one contiguous
// range of logical tiles, so tiles that share operand rows meet in the same L2.
__device__ inline int xcd_contiguous(int hw_id, int total) {
  const int xcd = hw_id & 7, slot = hw_id >> 3;
  const int base = total >> 3, rem = total & 7;
  return xcd * base + (xcd < rem ? xcd : rem) + slot;
}

// Raw buffer descriptor over a tensor: loads whose byte offset is >= `bytes` return zero without
// touching memory, which is how padding pixels, ragged tile rows and channel tails are filled.
__device__ inline __amdgpu_buffer_rsrc_t make_rsrc(const void *p, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, 0x00020000);
}
constexpr unsigned kOOB = 0x80000000u;   // every tensor is smaller than 2 GiB (checked on the host)

__device__ inline f32x4 buffer_load_16B(__amdgpu_buffer_rsrc_t r, unsigned voff) {
  return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)voff, 0, 0));
}

// Epilogue of a BM x BN output tile.  put_tile() writes the accumulators to Cs (fp32 [BM][BN + 8] in LDS, which must
// be free); from there global memory sees 16-byte accesses along the channel axis.  row_off: per tile row the index
// of its output pixel, -1 past the end.  The optional addend is added in fp32 before the one rounding to T.
template <typename T, int BM, int BN, int NT, int MODE, typename PutTile>
__device__ inline void conv_epilogue(const ArgsOf<MODE> &a, float (*Cs)[BN + 8], const int *row_off, int tm, int n0, PutTile put_tile) {
  using E = Elem<T>;
  constexpr int VEC = E::VEC;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  T *out = static_cast<T *>(a.out);
  const T *addend = static_cast<const T *>(a.addend);
  constexpr int CV = BN / VEC;            // 16-byte pieces per tile row
  constexpr bool kSpare = NT / CV > BM;   // a tile with fewer pieces than there are threads
  constexpr int RPS = kSpare ? BM : NT / CV;      // rows per pass
  constexpr int NP = BM / RPS;      // passes over the tile
  constexpr int PG = NP < 8 ? NP : 8;   // passes whose side inputs are in flight together
  static_assert(BM % RPS == 0 && CV <= 32 && NP % PG == 0, "output tile rows per pass");
  const int cv = (tid % CV) * VEC, row0 = tid / CV;
  const bool col_ok = n0 + cv < a.OC;     // OC is a multiple of VEC
  const bool bn_bwd = MODE == kBwd && a.bn_sums != nullptr;
  // The side inputs of the epilogue (addend, ReLU mask, BN input: up to three 16-byte loads per thread
  // and pass) are requested for up to eight passes at once, the first group here, before the
  // accumulators even go to LDS: taken one pass at a time, every pass would wait out a memory round
  // trip of its own (a store to `out` may alias the addend, so the compiler cannot move the loads
  // itself).  A thread reads only elements it writes later.
  const T *maskp = static_cast<const T *>(a.relu_mask), *bnyp = static_cast<const T *>(a.bn_y);
  const bool has_mask = MODE == kBwd && a.relu_mask != nullptr;
  typename Vec<T>::Raw q_ad[PG], q_mk[PG], q_y[PG];
  size_t offs[PG];
  bool live[PG];
  auto request_side = [&](int p0) {
#pragma unroll
    for (int g = 0; g < PG; ++g) {
      int ro = -1;
      if (!kSpare || row0 < BM) ro = row_off[row0 + (p0 + g) * RPS];
      live[g] = ro >= 0 && col_ok;
      offs[g] = live[g] ? (size_t)ro * a.OC + n0 + cv : 0;
      q_ad[g] = q_mk[g] = q_y[g] = typename Vec<T>::Raw{};
      if (live[g]) {
        if (addend) q_ad[g] = Vec<T>::load_raw(addend + offs[g]);
        if (has_mask) q_mk[g] = Vec<T>::load_raw(maskp + offs[g]);
        if (bn_bwd) q_y[g] = Vec<T>::load_raw(bnyp + offs[g]);
        if constexpr (MODE == kEval) {
          if (a.act_res) q_y[g] = Vec<T>::load_raw(static_cast<const T *>(a.act_res) + offs[g]);
        }
      }
    }
  };
  request_side(0);
  put_tile();
  __syncthreads();
  // batch-norm statistics of this row tile: column sums of (v - k) and (v - k)^2 of the values v as
  // stored, with the shift k = the tile's first accumulated row of the column.  Any k within a few
  // standard deviations of the column keeps the sum of squares free of the cancellation that
  // sum(v^2) - (sum v)^2/n suffers when |mean| >> std.
  float s1[VEC], s2[VEC], kshift[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) { s1[e] = 0.f; s2[e] = 0.f; kshift[e] = 0.f; }
  float bmu[VEC], bis[VEC], bsc[VEC], bsh[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) { bmu[e] = 0.f; bis[e] = 0.f; bsc[e] = 0.f; bsh[e] = 0.f; }
  if (bn_bwd && col_ok) {
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
      const int c = n0 + cv + e;
      bmu[e] = a.bn_mean[c]; bis[e] = a.bn_invstd[c]; bsc[e] = a.bn_scale[c]; bsh[e] = a.bn_shift[c];
    }
  }
  if constexpr (MODE == kEval) {
    if (col_ok) {
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        const int c = n0 + cv + e;
        bsc[e] = a.act_scale[c]; bsh[e] = a.act_shift[c];
        bmu[e] = a.res_scale ? a.res_scale[c] : 1.f;
        bis[e] = a.res_scale ? a.res_shift[c] : 0.f;
      }
    }
  }
  if (MODE == kFwd && a.stats) {
#pragma unroll
    for (int e = 0; e < VEC; e += 4) {
      const f32x4 t = *reinterpret_cast<const f32x4 *>(&Cs[0][cv + e]);
      kshift[e] = t[0]; kshift[e + 1] = t[1]; kshift[e + 2] = t[2]; kshift[e + 3] = t[3];
    }
  }
#pragma unroll
  for (int p0 = 0; p0 < NP; p0 += PG) {
    if (p0 > 0) request_side(p0);
#pragma unroll
    for (int g = 0; g < PG; ++g) {
      if (!live[g]) continue;
      const int r = row0 + (p0 + g) * RPS;
      const size_t off = offs[g];
      float v[VEC];
#pragma unroll
      for (int e = 0; e < VEC; e += 4) {
        const f32x4 t = *reinterpret_cast<const f32x4 *>(&Cs[r][cv + e]);
        v[e] = t[0]; v[e + 1] = t[1]; v[e + 2] = t[2]; v[e + 3] = t[3];
      }
      if (addend) {
        float ad[VEC];
        Vec<T>::unpack(q_ad[g], ad);
#pragma unroll
        for (int e = 0; e < VEC; ++e) v[e] += ad[e];
      }
      if (has_mask) {
        float mk[VEC];
        Vec<T>::unpack(q_mk[g], mk);
#pragma unroll
        for (int e = 0; e < VEC; ++e) v[e] = mk[e] > 0.f ? v[e] : 0.f;
      }
      if (MODE != kEval || out) Vec<T>::store(out + off, v);
      if constexpr (MODE == kEval) {
        // the arithmetic of bn_apply_kernel on the value as stored
        float rv[VEC], o[VEC];
        if (a.act_res) Vec<T>::unpack(q_y[g], rv);
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
          o[e] = fmaf(E::to_f32(E::from_f32(v[e])), bsc[e], bsh[e]);
          if (a.act_res) o[e] += fmaf(rv[e], bmu[e], bis[e]);
          o[e] = o[e] > 0.f ? o[e] : 0.f;
        }
        Vec<T>::store(static_cast<T *>(a.act) + off, o);
      }
      if (bn_bwd) {
        // the same arithmetic as the stand-alone first pass (bn_bwd_partial_kernel) on the values as stored
        float yv[VEC];
        Vec<T>::unpack(q_y[g], yv);
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
          float gm = E::to_f32(E::from_f32(v[e]));
          if (a.bn_self) gm = fmaf(yv[e], bsc[e], bsh[e]) > 0.f ? gm : 0.f;
          const float xh = (yv[e] - bmu[e]) * bis[e];
          s1[e] += gm;
          s2[e] = fmaf(gm, xh, s2[e]);
        }
      }
      if (MODE == kFwd) {
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
          const float sv = E::to_f32(E::from_f32(v[e])) - kshift[e];
          s1[e] += sv;
          s2[e] = fmaf(sv, sv, s2[e]);
        }
      }
    }
  }
  if ((MODE == kFwd && a.stats) || bn_bwd) {
    // A wave holds 64/CV rows of every column piece: butterfly over those lanes, then the waves add
    // up in wave order.  Every step has a fixed order, so the sums are bit-stable from run to run.
    constexpr int NW = NT / 64;
    __shared__ float red[2][NW][BN];
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
#pragma unroll
      for (int o = CV; o < 64; o <<= 1) {
        s1[e] += __shfl_xor(s1[e], o, 64);
        s2[e] += __shfl_xor(s2[e], o, 64);
      }
    }
    if (lane < CV) {
#pragma unroll
      for (int e = 0; e < VEC; ++e) { red[0][wave][cv + e] = s1[e]; red[1][wave][cv + e] = s2[e]; }
    }
    __syncthreads();
    for (int c = tid; c < BN; c += NT) {
      if (n0 + c < a.OC) {
        float t1 = red[0][0][c], t2 = red[1][0][c];
#pragma unroll
        for (int w = 1; w < NW; ++w) { t1 += red[0][w][c]; t2 += red[1][w][c]; }
        if (MODE == kFwd) {
          a.stats[(size_t)tm * a.OC + n0 + c] = Cs[0][c];
          a.stats[((size_t)a.tiles_m + tm) * a.OC + n0 + c] = t1;
          a.stats[((size_t)2 * a.tiles_m + tm) * a.OC + n0 + c] = t2;
        } else {
          a.bn_sums[(size_t)tm * a.OC + n0 + c] = t1;
          a.bn_sums[((size_t)a.tiles_m + tm) * a.OC + n0 + c] = t2;
        }
      }
    }
  }
}

}  // namespace

// 3x3 stride-1 convolutions on filters in matrix fragments, in fp32 through operands split into three bf16 parts (conv3.hip)
bool conv3_takes(const IgemmArgs &a, int dt);
int64_t conv3_filter_bytes(int OC, int IC, int dt);
int conv3_launch(const EvalArgs &a, const Filter &w, int dt, int mode, hipStream_t st, StatParts *tiles_m_out);
int conv3_launch_rows(const EvalArgs &a, int mode, hipStream_t st, StatParts *tiles_m_out);   // fp32, on the filter's rows a.wt
// widening 1x1 convolutions in bf16, streamed (conv1.hip)
bool conv1_takes(const IgemmArgs &a, int dt, int mode);
int conv1_launch(const IgemmArgs &a, int mode, hipStream_t st, StatParts *tiles_m_out);
// convolutions with few output tiles: 32x32 tiles, the reduction split among the waves of a workgroup (conv_small.hip)
bool conv_small_takes(const IgemmArgs &a, int dt);
bool conv_small_rows(long long pixels, int OC, int cls);   // whether it may take an output of this size, in 32-row tiles
int conv_small_launch(const EvalArgs &a, int dt, int mode, hipStream_t st, StatParts *tiles_m_out);
int wgrad_tile(const ConvGeom &g);   // channels (square) a workgroup of the one-tap weight gradient takes
// the weight gradient of such a convolution (wgrad3.hip): out [splits][K][3][3][C], a multiple of 32 rows each
bool wgrad3_takes(const ConvGeom &g);
// the same in bf16, one filter row per workgroup
bool wgrad3_row_takes(const ConvGeom &g);
int wgrad3_row_launch(const ConvGeom &g, const void *dy, const void *x, float *out, int splits, int rows_per_split, hipStream_t st);
int wgrad3_launch(const ConvGeom &g, const float *dy, const float *x, float *out, int splits, int rows_per_split, hipStream_t st);

}  // namespace resist
