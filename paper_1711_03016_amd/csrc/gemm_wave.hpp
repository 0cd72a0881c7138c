// Dense-layer products whose waves load their matrix-core fragments straight
// from global memory and share the contraction between them.
//
// Same products and fused epilogues as gemm_kernel.hpp (NN forward, NT adjoint
// wrt the input, TN adjoint wrt the weights), float32 or bf16 operands. A workgroup
// of NW waves owns one tile of 16 AB x 16 BB outputs; every wave computes the whole
// tile over its own contiguous range of k-steps (16 k of float32, 32 of bf16), and
// the NW partial tiles are added in wave order through LDS at the end, where the
// epilogue runs.
//
// What bounds these products is not arithmetic: with a few hundred tiles each
// compute unit has one, and its time is the latency of reaching the operands.
// Staged through LDS, every k-stage cost a memory round trip and a barrier
// (about 3,500 cycles per 128 k of float32). Here the loads of DEPTH steps are in
// flight per wave, no barrier stands between the first load and the one reduction,
// and the operands cross no LDS. Measured back to back in float32 (rotating
// operands): 256 x 512 x 784 12.7 -> 5.8 us, 256 x 512 x 512 9.3 -> 4.3;
// 64 x 256 x 356 (a recurrent cell) 8.1 -> 3.3; 512 x 512 x 256 wrt the weights
// 6.8 -> 4.2. In bf16: 1000 x 500 x 784 (rows of 500) 45 -> 7.1, 4096 x 10 x 1024
// 11.3 -> 5.0, 1024 x 16 x 4096 wrt the weights 11.4 (in slices, with their sum) -> 7.3.
//
// Fragments without LDS. v_mfma_f32_16x16x4_f32 wants, in lane 16 g + l, the value
// of row (or column) l at the g-th of its 4 k; v_mfma_f32_16x16x32_bf16 the 8
// values at k = 8 g .. 8 g + 7. Both operands may use any assignment of k to
// (instruction, g) as long as they use the same one, and rows may be assigned to
// lanes in any order that the store undoes, so:
//   k-contiguous operand: one 16-byte load per 16-row block, lane (g, l) taking
//     the 4 (8) k at 4 g (8 g) of row l; float32 value e feeds instruction e.
//   row-contiguous operand (its k strided in memory): for each e of those k one
//     load of the 16 R columns of that k's row, lane l taking columns
//     R l .. R l + R - 1 (R = AB or BB); value i belongs to block i, whose row l is
//     thus row R l + i of the tile. bf16 values of consecutive k are paired by byte
//     permutes when they are multiplied.
// Loads go through a descriptor or base that moves with the step (scalar work) and
// byte offsets inside a step that each lane computes once. They ask for the
// alignment of one element only, so every leading dimension and size takes this
// path. Rows past the edge of the output are read from one inside (they reach only
// outputs that are not stored); a load of R columns that would straddle that edge
// starts R columns before it, and its values move into place when they are multiplied.
// In the k-step that crosses the end of the contraction (and in operands of fewer
// than R columns) values are loaded one by one, with an offset past the descriptor's
// size (the hardware returns zero) for what lies outside.
#pragma once

#include "common.hpp"
#include "gemm_kernel.hpp"
#include "kernels.hpp"

namespace dlvm {
namespace gemm {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr uint32_t kBufSize = 0x7fffff00u;  // bytes past a descriptor's base that offsets may reach
constexpr uint32_t kBufOut = 0x80000000u;   // an offset outside every descriptor: reads zero

template <typename T> constexpr int wave_step() { return sizeof(T) == 4 ? 16 : 32; }  // k of one step

__device__ __forceinline__ __amdgpu_buffer_rsrc_t wave_rsrc(const void* base) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0,
                                           static_cast<int>(kBufSize), 0x00020000);
}

// R consecutive floats at byte offset `off` of the descriptor.
template <int R>
__device__ __forceinline__ void buf_load(float (&d)[R], __amdgpu_buffer_rsrc_t rs, uint32_t off) {
  if constexpr (R == 4) {
    const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rs, static_cast<int>(off), 0, 0);
#pragma unroll
    for (int e = 0; e < 4; ++e) d[e] = __uint_as_float(v[e]);
  } else if constexpr (R == 2) {
    const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(rs, static_cast<int>(off), 0, 0);
    d[0] = __uint_as_float(v[0]);
    d[1] = __uint_as_float(v[1]);
  } else {
    static_assert(R == 1, "1, 2 or 4 floats");
    d[0] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, static_cast<int>(off), 0, 0));
  }
}

// One operand of a tile: R blocks of 16 rows. KMAJ: P[r * ld + k]; else P[k * ld + r].
// Lane (g, l) loads the E values at k = E g .. of a step.
template <typename T, bool KMAJ, int R>
struct WaveOffsets {
  static constexpr int E = wave_step<T>() / 4;
  uint32_t off[KMAJ ? R : E];  // byte offsets inside a step from the tile's origin
  int ahead = 0;               // columns by which this lane's loads start early
  int back = 0;                // columns before the tile's origin where the loads' base lies

  // Rows past `rows` (rows left in the operand from the tile's first) are read
  // from one inside: they only reach outputs that are not stored.
  __device__ __forceinline__ void init(int64_t ld, int lane, int64_t rows) {
    const int l = lane & 15, g = lane >> 4;
    if constexpr (!KMAJ && R > 1) back = rows < R ? static_cast<int>(R - rows) : 0;
#pragma unroll
    for (int i = 0; i < (KMAJ ? R : E); ++i) {
      if constexpr (KMAJ) {
        const int64_t r = 16 * i + l < rows ? 16 * i + l : 0;
        off[i] = static_cast<uint32_t>((r * ld + E * g) * static_cast<int64_t>(sizeof(T)));
      } else {
        const int64_t r = R * l >= rows ? 0 : R * l + R <= rows ? R * l : rows - R + back;
        off[i] = static_cast<uint32_t>(((E * g + i) * ld + r) * static_cast<int64_t>(sizeof(T)));
      }
    }
    if constexpr (!KMAJ && R > 1)
      ahead = R * l < rows && R * l + R > rows ? static_cast<int>(R * l + R - rows) : 0;
  }
  // Byte offset of value e of block i, or one outside every descriptor where
  // the row lies past `rows` or its k past `ks` (counted from the origin).
  __device__ __forceinline__ static uint32_t edge(int i, int e, int64_t ld, int lane, int64_t rows,
                                                  int64_t ks) {
    const int l = lane & 15, g = lane >> 4;
    const int r = KMAJ ? 16 * i + l : R * l + i, k = E * g + e;
    const int64_t o = (KMAJ ? r * ld + k : k * ld + r) * static_cast<int64_t>(sizeof(T));
    return r < rows && k < ks ? static_cast<uint32_t>(o) : kBufOut;
  }
};

template <typename T, bool KMAJ, int R> struct WaveOperand;

// float32: value e of block i feeds instruction e of the step.
template <bool KMAJ, int R>
struct WaveOperand<float, KMAJ, R> : WaveOffsets<float, KMAJ, R> {
  struct Regs { float v[4][R]; };
  using WaveOffsets<float, KMAJ, R>::off;

  // The step whose first k lies at `P` (the tile's origin row), all inside the operand.
  __device__ __forceinline__ void load(Regs& f, const float* P) const {
    const __amdgpu_buffer_rsrc_t rs = wave_rsrc(P - this->back);
    if constexpr (KMAJ) {
#pragma unroll
      for (int i = 0; i < R; ++i) {
        float t[4];
        buf_load<4>(t, rs, off[i]);
#pragma unroll
        for (int e = 0; e < 4; ++e) f.v[e][i] = t[e];
      }
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) buf_load<R>(f.v[e], rs, off[e]);
    }
  }
  // The values of loads that started early, in their places (those past the edge are
  // anything: they reach only outputs that are not stored).
  __device__ __forceinline__ Regs settled(const Regs& f) const {
    Regs o;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if constexpr (KMAJ || R == 1) {
#pragma unroll
        for (int i = 0; i < R; ++i) o.v[e][i] = f.v[e][i];
      } else if constexpr (R == 2) {
        o.v[e][0] = this->ahead ? f.v[e][1] : f.v[e][0];
        o.v[e][1] = f.v[e][1];
      } else {
        const float x0 = (this->ahead & 2) ? f.v[e][2] : f.v[e][0];
        const float x1 = (this->ahead & 2) ? f.v[e][3] : f.v[e][1];
        o.v[e][0] = (this->ahead & 1) ? x1 : x0;
        o.v[e][1] = (this->ahead & 1) ? f.v[e][2] : x1;
        o.v[e][2] = (this->ahead & 1) ? f.v[e][3] : f.v[e][2];
        o.v[e][3] = f.v[e][3];
      }
    }
    return o;
  }
  // The same value by value, zeros for rows from `rows` and k from `ks` on.
  __device__ __forceinline__ void load_edge(Regs& f, const float* P, int64_t ld, int lane,
                                            int64_t rows, int64_t ks) const {
    const __amdgpu_buffer_rsrc_t rs = wave_rsrc(P);
#pragma unroll
    for (int i = 0; i < R; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float t[1];
        buf_load<1>(t, rs, this->edge(i, e, ld, lane, rows, ks));
        f.v[e][i] = t[0];
      }
  }
};

// bf16: k-contiguous, the 8 values of block i in v[i]; row-contiguous, the R values
// at each k in w[e] (two to a word).
template <bool KMAJ, int R>
struct WaveOperand<bf16_t, KMAJ, R> : WaveOffsets<bf16_t, KMAJ, R> {
  static constexpr int W = R > 1 ? R / 2 : 1;
  struct Regs { uint32_t w[KMAJ ? R : 8][KMAJ ? 4 : W]; };
  using WaveOffsets<bf16_t, KMAJ, R>::off;
  struct __attribute__((packed, aligned(2))) Words { uint32_t w[KMAJ ? 4 : W]; };

  __device__ __forceinline__ void load(Regs& f, const bf16_t* P) const {
    const char* const base = reinterpret_cast<const char*>(P - this->back);
#pragma unroll
    for (int i = 0; i < (KMAJ ? R : 8); ++i) {
      if constexpr (!KMAJ && R == 1) {
        f.w[i][0] = *reinterpret_cast<const bf16_t*>(base + off[i]);
      } else {
        const Words t = *reinterpret_cast<const Words*>(base + off[i]);
#pragma unroll
        for (int q = 0; q < (KMAJ ? 4 : W); ++q) f.w[i][q] = t.w[q];
      }
    }
  }
  __device__ __forceinline__ void load_edge(Regs& f, const bf16_t* P, int64_t ld, int lane,
                                            int64_t rows, int64_t ks) const {
    const __amdgpu_buffer_rsrc_t rs = wave_rsrc(P);
    auto one = [&](int i, int e) {
      return static_cast<uint32_t>(static_cast<uint16_t>(__builtin_amdgcn_raw_buffer_load_b16(
          rs, static_cast<int>(this->edge(i, e, ld, lane, rows, ks)), 0, 0)));
    };
    if constexpr (KMAJ) {
#pragma unroll
      for (int i = 0; i < R; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) f.w[i][q] = one(i, 2 * q) | (one(i, 2 * q + 1) << 16);
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        if constexpr (R == 1) {
          f.w[e][0] = one(0, e);
        } else {
#pragma unroll
          for (int q = 0; q < W; ++q) f.w[e][q] = one(2 * q, e) | (one(2 * q + 1, e) << 16);
        }
      }
    }
  }
  __device__ __forceinline__ Regs settled(const Regs& f) const {
    Regs o;
#pragma unroll
    for (int e = 0; e < (KMAJ ? R : 8); ++e) {
      if constexpr (KMAJ) {
#pragma unroll
        for (int q = 0; q < 4; ++q) o.w[e][q] = f.w[e][q];
      } else if constexpr (R == 4) {
        const uint64_t x = ((static_cast<uint64_t>(f.w[e][1]) << 32) | f.w[e][0]) >> (16 * this->ahead);
        o.w[e][0] = static_cast<uint32_t>(x);
        o.w[e][1] = static_cast<uint32_t>(x >> 32);
      } else {
        o.w[e][0] = R == 2 ? f.w[e][0] >> (16 * this->ahead) : f.w[e][0];
      }
    }
    return o;
  }
  // The 8 values of block i.
  __device__ __forceinline__ static bf16x8 frag(const Regs& f, int i) {
    if constexpr (KMAJ) {
      return __builtin_bit_cast(bf16x8, make_uint4(f.w[i][0], f.w[i][1], f.w[i][2], f.w[i][3]));
    } else {
      uint32_t t[4];
#pragma unroll
      for (int q = 0; q < 4; ++q)
        t[q] = perm_b32(f.w[2 * q + 1][i >> 1], f.w[2 * q][i >> 1], (i & 1) ? 0x07060302u : 0x05040100u);
      return __builtin_bit_cast(bf16x8, make_uint4(t[0], t[1], t[2], t[3]));
    }
  }
};

// LDS bytes of one workgroup: the waves' partial tiles (rows padded by 16
// bytes: the stores of a wave's four row groups fall into different banks) and
// the partial column sums.
template <int AB, int BB, int NW>
constexpr int wave_smem_bytes() {
  return NW * (16 * AB * (16 * BB + 4) + 16 * BB) * 4;
}

// Softmax cross-entropy of a tile's 16 rows of logits (EPI_XENT; see Params::C2):
// thread TN r + c takes column c of row r, so a row is 16 or 32 neighbouring lanes.
// The partial products are summed here (with the bias `b`), so neither the logits
// nor their slices cross memory between the output layer and its loss. Measured on
// 10 classes, the sliced product and its loss before and this launch now: 256 rows of
// 512 float32 6.8 + 4.6 -> 5.3 us; 4096 rows of 1024 bf16 7.4 + 4.2 -> 6.3.
template <typename T, int TN, int NW>
__device__ __forceinline__ void wave_xent(const Params& p, const float* part, float* rowv, int ld,
                                          int64_t m0, int tile, int tid, float b) {
  constexpr int TM = 16;
  const int r = tid / TN, c = tid % TN;
  const int64_t row = m0 + r;
  const bool in = tid < TM * TN, live = in && row < p.M, valid = live && c < p.N;
  float z = 0.0f;
  if (in) {
    z = part[r * ld + c];
#pragma unroll
    for (int w = 1; w < NW; ++w) z += part[w * TM * ld + r * ld + c];
    z = p.alpha * z + b;
  }
  const int y = live ? static_cast<const int32_t*>(p.aux)[row] : 0;
  const bool ok = y >= 0 && y < p.N;
  float m = row16_max(valid ? z : -INFINITY);
  if constexpr (TN == 32) m = fmaxf(m, __shfl_xor(m, 16, 64));
  const float e = valid ? __expf(z - m) : 0.0f;
  float s = row16_sum(e), zy = row16_sum(valid && c == y ? z : 0.0f);  // (one term: exact)
  if constexpr (TN == 32) {
    s += __shfl_xor(s, 16, 64);
    zy += __shfl_xor(zy, 16, 64);
  }
  if (live && c < p.lda2) {
    const float d = valid ? p.inv_n / s * e - (c == y ? p.inv_n : 0.0f) : 0.0f;
    static_cast<T*>(p.C2)[row * p.lda2 + c] = store_cast<T>(d);
  }
  if (valid && p.C != nullptr) static_cast<float*>(p.C)[row * p.ldc + c] = z;
  if (in && c == 0) {
    rowv[r] = !live ? 0.0f : ok ? (m + __logf(s)) - zy : NAN;
    reinterpret_cast<int*>(rowv)[TM + r] = live && !ok ? 1 : 0;
  }
  __syncthreads();
  if (tid == 0) {
    float t = 0.0f;
    int bad = 0;
#pragma unroll
    for (int q = 0; q < TM; ++q) {
      t += rowv[q];
      bad += reinterpret_cast<const int*>(rowv)[TM + q];
    }
    p.partials[tile] = t;
    static_cast<int32_t*>(const_cast<void*>(p.residual))[tile] = bad;
  }
}

// One output tile (`tile` from split_slice) of a product, LDS at `smem`. EDGE:
// the tile crosses the edge of the output; ONE: a row-contiguous operand has fewer
// columns in all than one load takes, so values are loaded one by one.
template <typename T, typename TO, bool AK, bool BKM, int AB, int BB, int NW, int DEPTH, int EPI,
          bool PH2, bool EDGE, bool ONE>
__device__ __forceinline__ void wave_gemm_body(const Params& p, int64_t m0, int64_t n0, int tm,
                                               int tile, char* smem) {
  constexpr int TM = 16 * AB, TN = 16 * BB, LD = TN + 4;
  constexpr int THREADS = 64 * NW, STEP = wave_step<T>();
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l = lane & 15, g = lane >> 4;
  float* const part = reinterpret_cast<float*>(smem);          // [NW][TM][LD]
  float* const cpart = part + NW * TM * LD;                    // [NW][TN]

  // Outputs of this thread: element tid + j * THREADS of the tile, row by row.
  // What their epilogue reads is loaded now, behind the contraction.
  constexpr int PER = (TM * TN + THREADS - 1) / THREADS;
  static_assert(TM * TN % THREADS == 0 || PER == 1, "whole outputs per thread, or at most one");
  constexpr bool AHEAD = PER <= 2;
  float pre_b[AHEAD ? PER : 1], pre_g[AHEAD ? PER : 1], pre_r[AHEAD ? PER : 1];
  const T* const aux = static_cast<const T*>(p.aux);
  const TO* const res = static_cast<const TO*>(p.residual);
  const T* const bias = static_cast<const T*>(p.bias);
  const bool use_aux = EPI == EPI_CHAIN || (EPI == EPI_DACT && p.act != ACT_NONE);
  const bool use_res = EPI == EPI_DACT && res != nullptr;
  auto fetch = [&](int j, float& b, float& gr, float& r) {
    const int o = tid + j * THREADS;
    const int64_t row = m0 + o / TN, col = n0 + o % TN;
    const bool in = o < TM * TN && (!EDGE || (row < p.M && col < p.N));
    constexpr bool BIAS = EPI == EPI_STORE || EPI == EPI_CHAIN || EPI == EPI_XENT;
    b = BIAS && bias != nullptr && in && col < p.nvec ? load_as_f32<T>(bias + col) : 0.0f;
    gr = use_aux && in ? load_as_f32<T>(aux + row * p.ldc + col) : 0.0f;
    r = use_res && in ? load_as_f32<TO>(res + row * p.ldc + col) : 0.0f;
  };
  if constexpr (AHEAD) {
#pragma unroll
    for (int j = 0; j < PER; ++j) fetch(j, pre_b[j], pre_g[j], pre_r[j]);
  }

  // Steps: the whole ones of both phases in order, shared out over the waves;
  // what is left goes to the first wave, which never has more steps than another (of
  // two phases: what is left of the second to the last wave).
  const int64_t K1 = PH2 ? p.K1 : p.K;
  const int nf1 = static_cast<int>(K1 / STEP);
  const int nf = PH2 ? nf1 + static_cast<int>((p.K - K1) / STEP) : nf1;
  const int s0 = static_cast<int>(static_cast<int64_t>(nf) * wave / NW);
  const int s1 = static_cast<int>(static_cast<int64_t>(nf) * (wave + 1) / NW);
  const int64_t tail1 = PH2 ? K1 - static_cast<int64_t>(nf1) * STEP : 0;
  const int64_t tail2 = PH2 ? p.K - K1 - static_cast<int64_t>(nf - nf1) * STEP
                            : p.K - static_cast<int64_t>(nf) * STEP;

  // Origin of a step: the tile's first row (or column) at its first k.
  const T* const A = static_cast<const T*>(p.A);
  const T* const B = static_cast<const T*>(p.B);
  const T* const A2 = static_cast<const T*>(p.A2);
  auto a_at = [&](int s, int64_t& ld) {
    const bool ph2 = PH2 && s >= nf1;
    ld = ph2 ? p.lda2 : p.lda;
    const T* a = ph2 ? A2 : A;
    const int64_t k = static_cast<int64_t>(ph2 ? s - nf1 : s) * STEP;
    return AK ? a + m0 * ld + k : a + k * ld + m0;
  };
  auto b_at = [&](int s) {
    const int64_t k = PH2 && s >= nf1 ? K1 + static_cast<int64_t>(s - nf1) * STEP
                                      : static_cast<int64_t>(s) * STEP;
    return BKM ? B + n0 * p.ldb + k : B + k * p.ldb + n0;
  };

  using OA = WaveOperand<T, AK, AB>;
  using OB = WaveOperand<T, BKM, BB>;
  OA oa, oa2;
  OB ob;
  const int64_t rows_a = EDGE ? p.M - m0 : TM, rows_b = EDGE ? p.N - n0 : TN;
  oa.init(p.lda, lane, rows_a);
  if constexpr (PH2) oa2.init(p.lda2, lane, rows_a);
  ob.init(p.ldb, lane, rows_b);

  // float32: instruction e of a step adds to accumulator e % ACC, summed in pairs at the
  // end. These tiles take products that larger tiles would split over k, so four sums per
  // wave keep a sum as short as theirs (1000 terms: 1.1e-7 of the norm, 2.1e-7 with one
  // per wave). Larger tiles have no registers for it (136 on 2 x 2 blocks: one workgroup
  // per compute unit), and the steps of a recurrence, one after the other, are better
  // without the additions (48 launches 137 us, 139 with them; their sums are short).
  constexpr int ACC = sizeof(T) == 4 && AB * BB <= 2 && !PH2 ? 4 : 1;
  f32x4 accs[ACC][AB][BB];
#pragma unroll
  for (int q = 0; q < ACC; ++q)
#pragma unroll
    for (int i = 0; i < AB; ++i)
#pragma unroll
      for (int j = 0; j < BB; ++j) accs[q][i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  float cs[BB];
#pragma unroll
  for (int j = 0; j < BB; ++j) cs[j] = 0.0f;
  const bool do_colsum = EPI == EPI_DW && p.colsum != nullptr && tm == 0;

  typename OA::Regs a[DEPTH];
  typename OB::Regs b[DEPTH];
  auto load = [&](int d, int s) {
    int64_t ld;
    const T* pa = a_at(s, ld);
    if constexpr (ONE)
      oa.load_edge(a[d], pa, ld, lane, p.M - m0, STEP);
    else if (PH2 && s >= nf1)
      oa2.load(a[d], pa);
    else
      oa.load(a[d], pa);
    if constexpr (ONE)
      ob.load_edge(b[d], b_at(s), p.ldb, lane, p.N - n0, STEP);
    else
      ob.load(b[d], b_at(s));
  };
  auto products = [&](const typename OA::Regs& ra, const typename OB::Regs& rb) {
    if constexpr (sizeof(T) == 4) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < AB; ++i)
#pragma unroll
          for (int j = 0; j < BB; ++j)
            accs[e % ACC][i][j] =
                __builtin_amdgcn_mfma_f32_16x16x4f32(ra.v[e][i], rb.v[e][j], accs[e % ACC][i][j], 0, 0, 0);
      if constexpr (EPI == EPI_DW) {
        if (do_colsum) {
#pragma unroll
          for (int j = 0; j < BB; ++j) cs[j] += (rb.v[0][j] + rb.v[1][j]) + (rb.v[2][j] + rb.v[3][j]);
        }
      }
    } else {
      bf16x8 fa[AB], fb[BB];
#pragma unroll
      for (int i = 0; i < AB; ++i) fa[i] = OA::frag(ra, i);
#pragma unroll
      for (int j = 0; j < BB; ++j) fb[j] = OB::frag(rb, j);
#pragma unroll
      for (int i = 0; i < AB; ++i)
#pragma unroll
        for (int j = 0; j < BB; ++j)
          accs[0][i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[i], fb[j], accs[0][i][j], 0, 0, 0);
      if constexpr (EPI == EPI_DW) {
        if (do_colsum) {
#pragma unroll
          for (int j = 0; j < BB; ++j) {
            const uint4 x = __builtin_bit_cast(uint4, fb[j]);
            const uint32_t q[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
            for (int e = 0; e < 4; ++e)
              cs[j] += __uint_as_float(q[e] << 16) + __uint_as_float(q[e] & 0xffff0000u);
          }
        }
      }
    }
  };

  auto multiply = [&](int d) {
    if constexpr (EDGE && !ONE)
      products(oa.settled(a[d]), ob.settled(b[d]));
    else
      products(a[d], b[d]);
  };

  // A partial step (fewer k left of a phase than a step has), its loads first of all.
  const bool t1 = PH2 && tail1 > 0 && wave == 0;
  const bool t2 = tail2 > 0 && wave == (PH2 ? NW - 1 : 0);
  typename OA::Regs ta;
  typename OB::Regs tb;
  if (t1 || t2) {
    const int64_t k = t1 ? static_cast<int64_t>(nf1) * STEP
                         : static_cast<int64_t>(PH2 ? nf - nf1 : nf) * STEP;
    const bool second = PH2 && t2;
    const int64_t ld = second ? p.lda2 : p.lda, kb = second ? K1 + k : k;
    const T* src = second ? A2 : A;
    const int64_t left = t1 ? tail1 : tail2;
    oa.load_edge(ta, AK ? src + m0 * ld + k : src + k * ld + m0, ld, lane, p.M - m0, left);
    ob.load_edge(tb, BKM ? B + n0 * p.ldb + kb : B + kb * p.ldb + n0, p.ldb, lane, p.N - n0, left);
  }

  if (s1 > s0) {
    // (past the wave's last step the last one is loaded again: a static number of loads in flight)
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) load(d, s0 + d < s1 ? s0 + d : s1 - 1);
    __builtin_amdgcn_sched_barrier(0);
    int s = s0;
    for (; s + DEPTH < s1; s += DEPTH) {
#pragma unroll
      for (int d = 0; d < DEPTH; ++d) {
        multiply(d);
        load(d, s + d + DEPTH < s1 ? s + d + DEPTH : s1 - 1);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int d = 0; d < DEPTH; ++d)
      if (s + d < s1) multiply(d);
  }
  if (t1 || t2) products(ta, tb);

#pragma unroll
  for (int h = ACC / 2; h >= 1; h /= 2)
#pragma unroll
    for (int q = 0; q < h; ++q)
#pragma unroll
      for (int i = 0; i < AB; ++i)
#pragma unroll
        for (int j = 0; j < BB; ++j) accs[q][i][j] += accs[q + h][i][j];
  const f32x4 (&acc)[AB][BB] = accs[0];

  // Partial tiles to LDS in row-major order. Accumulator register r of block
  // (i, j) holds the block's row 4 g + r and column l.
  float* const mine = part + wave * TM * LD;
#pragma unroll
  for (int i = 0; i < AB; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = AK ? 16 * i + 4 * g + r : AB * (4 * g + r) + i;
      if constexpr (BKM || BB == 1) {
#pragma unroll
        for (int j = 0; j < BB; ++j) mine[row * LD + 16 * j + l] = acc[i][j][r];
      } else if constexpr (BB == 2) {
        *reinterpret_cast<float2*>(mine + row * LD + 2 * l) = make_float2(acc[i][0][r], acc[i][1][r]);
      } else {
        *reinterpret_cast<float4*>(mine + row * LD + 4 * l) =
            make_float4(acc[i][0][r], acc[i][1][r], acc[i][2][r], acc[i][3][r]);
      }
    }
  if constexpr (EPI == EPI_DW) {
    if (do_colsum) {
      // the four k groups of the wave (fixed order), then the waves below
#pragma unroll
      for (int j = 0; j < BB; ++j) {
        cs[j] += __shfl_xor(cs[j], 16, 64);
        cs[j] += __shfl_xor(cs[j], 32, 64);
        if (g == 0) cpart[wave * TN + (BKM ? 16 * j + l : BB * l + j)] = cs[j];
      }
    }
  }
  __syncthreads();

  TO* const C = static_cast<TO*>(p.C);
  if constexpr (EPI == EPI_XENT) {
    static_assert(AB == 1 && BB <= 2 && AHEAD && TM * TN <= THREADS, "one output per thread, rows of 16 or 32 lanes");
    wave_xent<T, TN, NW>(p, part, cpart, LD, m0, tile, tid, pre_b[0]);
    return;
  }
  float sq = 0.0f;  // EPI_CHAIN: this thread's sum of e^2
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int o = tid + j * THREADS;
    if (PER == 1 && o >= TM * TN) break;
    const int rr = o / TN, cc = o % TN;
    const int64_t row = m0 + rr, col = n0 + cc;
    float v = part[rr * LD + cc];
#pragma unroll
    for (int w = 1; w < NW; ++w) v += part[w * TM * LD + rr * LD + cc];
    if (EDGE && (row >= p.M || col >= p.N)) continue;
    float bv, gv, rv;
    if constexpr (AHEAD) {
      bv = pre_b[j]; gv = pre_g[j]; rv = pre_r[j];
    } else {
      fetch(j, bv, gv, rv);
    }
    if constexpr (EPI == EPI_CHAIN) {
      float xb, e;
      sq += chain_elem(v, bv, gv, p.inv_n, false, v, xb, e);
      static_cast<float*>(p.C2)[row * p.ldc + col] = xb;
    } else if constexpr (EPI == EPI_STORE) {
      v = apply_act(p.act, p.alpha * v + bv);
    } else if constexpr (EPI == EPI_DACT) {
      if (p.res_pre) v += rv;
      if (use_aux) v *= act_grad_from_output(p.act, gv);
      if (!p.res_pre) v += rv;
    }
    C[row * p.ldc + col] = store_cast<TO>(v);
  }
  if constexpr (EPI == EPI_CHAIN) {
    // one loss partial per tile: butterflies, then the waves in order
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) sq += __shfl_xor(sq, o, 64);
    if (lane == 0) cpart[wave] = sq;
    __syncthreads();
    if (tid == 0) {
      float t = cpart[0];
#pragma unroll
      for (int w = 1; w < NW; ++w) t += cpart[w];
      p.partials[tile] = t;
    }
  }
  if constexpr (EPI == EPI_DW) {
    if (do_colsum && tid < TN && n0 + tid < p.nvec) {
      float t = cpart[tid];
#pragma unroll
      for (int w = 1; w < NW; ++w) t += cpart[w * TN + tid];
      p.colsum[n0 + tid] = t;
    }
  }
}

template <typename T, typename TO, bool AK, bool BKM, int AB, int BB, int NW, int DEPTH, int EPI,
          bool PH2 = false>
__device__ __forceinline__ void wave_gemm_tile(const Params& p, int tile, char* smem) {
  int tm, tn;
  tile_of(tile, p.tiles_m, p.tiles_n, tm, tn);
  const int64_t m0 = static_cast<int64_t>(tm) * (16 * AB);
  const int64_t n0 = static_cast<int64_t>(tn) * (16 * BB);
  if (m0 + 16 * AB <= p.M && n0 + 16 * BB <= p.N) {
    wave_gemm_body<T, TO, AK, BKM, AB, BB, NW, DEPTH, EPI, PH2, false, false>(p, m0, n0, tm, tile, smem);
  } else {
    constexpr bool CA = !AK && AB > 1, CB = !BKM && BB > 1;  // loads of several columns
    // (a tile with fewer columns left than a load takes loads from the tile before: bf16
    // 659 x 321 x 192, one column left, 7.5 us, as 320 columns; value by value 13.5)
    if ((CA && p.M < AB) || (CB && p.N < BB))
      wave_gemm_body<T, TO, AK, BKM, AB, BB, NW, DEPTH, EPI, PH2, true, CA || CB>(p, m0, n0, tm, tile, smem);
    else
      wave_gemm_body<T, TO, AK, BKM, AB, BB, NW, DEPTH, EPI, PH2, true, false>(p, m0, n0, tm, tile, smem);
  }
}

template <typename T, typename TO, bool AK, bool BKM, int AB, int BB, int NW, int DEPTH, int EPI,
          bool PH2>
__global__ __launch_bounds__(64 * NW) void dlvm_gemm_wave_kernel(Params p) {
  __shared__ __attribute__((aligned(16))) char smem[wave_smem_bytes<AB, BB, NW>()];
  const int tile = split_slice<T, AK, BKM>(p, static_cast<int>(blockIdx.x));
  // (a k-slice of a split two-phase product lies in one phase)
  if (PH2 && p.splits <= 1)
    wave_gemm_tile<T, TO, AK, BKM, AB, BB, NW, DEPTH, EPI, PH2>(p, tile, smem);
  else
    wave_gemm_tile<T, TO, AK, BKM, AB, BB, NW, DEPTH, EPI, false>(p, tile, smem);
}

// The two adjoint products of one dense layer in one launch (blocks [0, n1):
// TN wrt the weights, the rest: NT wrt the input), as dlvm_gemm_pair_kernel;
// the two may use different tiles.
template <typename T, typename TO2, int AB1, int BB1, int D1, int AB2, int BB2, int D2, int NW>
__global__ __launch_bounds__(64 * NW) void dlvm_gemm_wave_pair_kernel(Params p1, Params p2, int n1) {
  constexpr int S1 = wave_smem_bytes<AB1, BB1, NW>(), S2 = wave_smem_bytes<AB2, BB2, NW>();
  __shared__ __attribute__((aligned(16))) char smem[S1 > S2 ? S1 : S2];
  const int b = static_cast<int>(blockIdx.x);
  if (b < n1) {
    const int tile = split_slice<T, false, false>(p1, b);
    wave_gemm_tile<T, float, false, false, AB1, BB1, NW, D1, EPI_DW>(p1, tile, smem);
  } else {
    const int tile = split_slice<T, true, true>(p2, b - n1);
    wave_gemm_tile<T, TO2, true, true, AB2, BB2, NW, D2, EPI_DACT>(p2, tile, smem);
  }
}

}  // namespace gemm
}  // namespace dlvm
