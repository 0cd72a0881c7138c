// Large float32 dense-layer products: tiles staged in LDS by direct-to-LDS
// loads (the same products and fused epilogues as gemm_kernel.hpp).
//
// Bound by the float32 matrix rate (157 TFLOP/s): one 32 x 32 x 2 instruction
// takes 64 cycles, so operand traffic is small beside it (a 128 x 128 tile
// reads 32 KiB for 4,096 cycles of every SIMD's matrix work) and what is lost
// is lost to waiting. Through registers, every k-tile cost address arithmetic, selects
// and LDS writes between two barriers, with the matrix cores idle for a fifth
// of the time. Here a wave's share of a k-tile is a few direct loads issued
// before its matrix work, into the other LDS slot, and a barrier per k-tile;
// two workgroups share a compute unit, so that one multiplies while the other
// waits. Measured (us, before and after, the same box): 8192 x 4096 x 4096 NN
// 2,181 -> 1,930 (142 TFLOP/s) and NT 2,219 -> 1,945, 4096 x 4096 x 8192 TN 2,260
// -> 1,880 (146); 2049 x 1001 x 777, whose rows are not 16-byte aligned, NN
// 95 -> 48. With neither loads nor barriers the loop reaches 144-149 TFLOP/s, so
// what is left of the gap to 157 is the wave's own issue of reads and instructions.
//
// LDS layouts (no padding), k-tiles of 32:
//   k-contiguous operand: rows of 128 bytes; the 16-byte chunk c of row r sits in
//     slot c ^ kswz(r), so a fragment read (lane l of half h takes 4 consecutive k
//     of row l, one per instruction) touches every bank evenly.
//   row-contiguous operand: k-rows of ROWS floats as in memory; instruction e of
//     step s wants row l at k = 8 s + 4 h + e: 32 consecutive floats per half.
//     The 128-byte column groups of k-rows with bit 2 of k set are exchanged in
//     pairs, so the two halves read different banks. No transpose is needed:
//     a lane's fragment is one float per instruction.
// VEC: 16 bytes per lane and load (16-byte aligned rows); else 4 bytes, which every
// float32 operand allows.
#pragma once

#include "common.hpp"
#include "gemm_async.hpp"
#include "gemm_kernel.hpp"
#include "kernels.hpp"

namespace dlvm {
namespace gemm {

constexpr int kF32Step = 32;  // k of one LDS k-tile

// This lane's place in the tile for wave instruction q of an operand tile of
// ROWS rows: the row and the k (of the first element it moves).
template <bool KMAJ, int ROWS, bool VEC>
__device__ __forceinline__ void f32_place(int q, int lane, int& r, int& k) {
  constexpr int W = VEC ? 4 : 1;             // floats per lane
  const int f = (q * 64 + lane) * W;         // first float of this lane inside the tile
  if constexpr (KMAJ) {
    r = f / kF32Step;
    const int slot = (f % kF32Step) >> 2;
    k = ((slot ^ kswz<64>(r)) << 2) + (f & 3);
  } else {
    k = f / ROWS;
    const int c = f % ROWS;
    r = c ^ (((k >> 2) & 1) << 5);
  }
}

// Direct loads of one k-tile of an operand into LDS: P is the tile's origin
// (its first row at the k-tile's first k); rows past `rows` are read from the
// last one (they only reach outputs that are not stored).
template <bool KMAJ, int ROWS, bool VEC, int NW>
struct F32Loader {
  static constexpr int W = VEC ? 4 : 1;
  static constexpr int N = ROWS * kF32Step / (64 * W) / NW;  // wave instructions per wave
  static_assert(ROWS * kF32Step % (64 * W * NW) == 0, "tile split over waves");
  uint32_t off[N];

  __device__ __forceinline__ static uint32_t offset(int r, int k, int64_t ld, int64_t rows) {
    int64_t rr = r;
    if constexpr (KMAJ) {
      rr = rr < rows ? rr : rows - 1;
      return static_cast<uint32_t>((rr * ld + k) * 4);
    } else {
      rr = rr < rows ? rr : 0;
      return static_cast<uint32_t>((k * ld + rr) * 4);
    }
  }
  __device__ __forceinline__ void init(int64_t ld, int64_t rows, int wave, int lane) {
#pragma unroll
    for (int j = 0; j < N; ++j) {
      int r, k;
      f32_place<KMAJ, ROWS, VEC>(wave * N + j, lane, r, k);
      off[j] = offset(r, k, ld, rows);
    }
  }
  __device__ __forceinline__ static void move(const __amdgpu_buffer_rsrc_t rs, char* lds, uint32_t o) {
    if constexpr (VEC)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, DLVM_LDS_PTR(lds), 16, o, 0, 0, 0);
    else
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, DLVM_LDS_PTR(lds), 4, o, 0, 0, 0);
  }
  __device__ __forceinline__ void load(const float* P, char* lds, int wave) const {
    const __amdgpu_buffer_rsrc_t rs = make_rsrc(P, 0x7fffff00u);
#pragma unroll
    for (int j = 0; j < N; ++j) move(rs, lds + (wave * N + j) * (256 * W), off[j]);
  }
  // The last k-tile of a phase, `kv` k of it valid: the rest is read from its
  // first k (and zeroed in LDS before use).
  __device__ __forceinline__ static void load_tail(const float* P, char* lds, int64_t ld,
                                                   int64_t rows, int kv, int wave, int lane) {
    const __amdgpu_buffer_rsrc_t rs = make_rsrc(P, 0x7fffff00u);
#pragma unroll
    for (int j = 0; j < N; ++j) {
      int r, k;
      f32_place<KMAJ, ROWS, VEC>(wave * N + j, lane, r, k);
      move(rs, lds + (wave * N + j) * (256 * W), offset(r, k < kv ? k : 0, ld, rows));
    }
  }
};

// Zero the k >= kv part of an operand tile.
template <bool KMAJ, int ROWS, int THREADS>
__device__ __forceinline__ void f32_zero_tail(char* lds, int kv, int tid) {
  float* const t = reinterpret_cast<float*>(lds);
  if constexpr (KMAJ) {
    for (int q = tid; q < ROWS * kF32Step; q += THREADS) {
      int r, k;
      f32_place<true, ROWS, false>(q >> 6, q & 63, r, k);
      if (k >= kv) t[q] = 0.0f;
    }
  } else {
    for (int q = kv * ROWS + tid; q < kF32Step * ROWS; q += THREADS) t[q] = 0.0f;
  }
}

// Fragment of the 32-row block at row0 for step s (8 k): f[e] feeds instruction e.
template <bool KMAJ, int ROWS>
__device__ __forceinline__ void f32_frag(float (&f)[4], const char* lds, int row0, int s, int lane) {
  if constexpr (KMAJ) {
    const int r = row0 + (lane & 31), c = 2 * s + (lane >> 5);
    const float4 v = *reinterpret_cast<const float4*>(lds + kmaj_off<64>(r, c));
    f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w;
  } else {
    const int h = lane >> 5;
    const int c = (row0 + (lane & 31)) ^ (h << 5);
    const float* p = reinterpret_cast<const float*>(lds) + (8 * s + 4 * h) * ROWS + c;
#pragma unroll
    for (int e = 0; e < 4; ++e) f[e] = p[e * ROWS];
  }
}

// Accumulators per output: instruction e of a step adds to accumulator e % ACC, and they
// are summed in pairs before the epilogue. A float32 sum's error grows with the root of
// its length (1000 terms: 5.7e-7 of the norm on one accumulator, 3.9e-7 on two, 2.8e-7 on
// four), and the tiles of few blocks have the registers for more than one. (The
// instructions of a wave with one block no longer wait for each other, which with two
// workgroups on a compute unit gains nothing: 2049 x 1001 x 777, all three products, 126 us
// either way.)
template <int TM, int TN> constexpr int f32_accs() { return TM * TN >= 4 ? 1 : 4 / (TM * TN); }

// One step (8 k) of the wave's TM x TN blocks: the matrix instructions of the
// fragments in register set CUR, with the reads of step s2 of the k-tile at
// (As2, Bs2) into the other set ahead of them. Consecutive instructions go to
// different accumulators (a dependent one would wait 8 cycles more).
template <bool AK, bool BKM, int BM, int BN, int TM, int TN, bool CS, int CUR>
__device__ __forceinline__ void f32_step(float (&a)[2][TM][4], float (&b)[2][TN][4],
                                         const char* __restrict__ As2, const char* __restrict__ Bs2,
                                         int s2, int arow, int brow, int lane,
                                         f32x16 (&acc)[f32_accs<TM, TN>()][TM][TN],
                                         float (&cs)[TN], bool do_cs) {
  constexpr int ACC = f32_accs<TM, TN>();
#pragma unroll
  for (int i = 0; i < TM; ++i) f32_frag<AK, BM>(a[CUR ^ 1][i], As2, arow + 32 * i, s2, lane);
#pragma unroll
  for (int j = 0; j < TN; ++j) f32_frag<BKM, BN>(b[CUR ^ 1][j], Bs2, brow + 32 * j, s2, lane);
#pragma unroll
  for (int e = 0; e < 4; ++e)
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
        acc[e % ACC][i][j] =
            __builtin_amdgcn_mfma_f32_32x32x2f32(a[CUR][i][e], b[CUR][j][e], acc[e % ACC][i][j], 0, 0, 0);
  // One instruction per block first: the set the reads go to feeds the
  // previous step's last instructions, which are then done with it. Then the
  // reads between the others (two per instruction).
  __builtin_amdgcn_sched_group_barrier(0x008, TM * TN, 0);
#pragma unroll
  for (int q = 0; q < 3 * TM * TN; ++q) {
    __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
  }
  __builtin_amdgcn_sched_barrier(0);
  if constexpr (CS) {
    if (do_cs) {
#pragma unroll
      for (int j = 0; j < TN; ++j) cs[j] += (b[CUR][j][0] + b[CUR][j][1]) + (b[CUR][j][2] + b[CUR][j][3]);
    }
  }
}

// One output tile (`tile` from split_slice), LDS ring of STAGES k-tiles at
// `smem` (1024-byte aligned).
template <bool AK, bool BKM, int BM, int BN, int WM, int WN, int STAGES, bool VEC, int EPI, bool PH2>
__device__ __forceinline__ void f32_gemm_tile(const Params& p, const int tile, char* smem) {
  constexpr int NW = WM * WN, THREADS = 64 * NW;
  constexpr int TM = BM / WM / 32, TN = BN / WN / 32;
  constexpr int A_BYTES = BM * kF32Step * 4, STAGE = (BM + BN) * kF32Step * 4;
  static_assert(AK || BM >= 64, "row-contiguous tile: whole pairs of column groups");
  static_assert(BKM || BN >= 64, "row-contiguous tile: whole pairs of column groups");
  using LA = F32Loader<AK, BM, VEC, NW>;
  using LB = F32Loader<BKM, BN, VEC, NW>;
  constexpr int LOADS = LA::N + LB::N;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  int tm, tn;
  tile_of(tile, p.tiles_m, p.tiles_n, tm, tn);
  const int64_t m0 = static_cast<int64_t>(tm) * BM, n0 = static_cast<int64_t>(tn) * BN;
  const int64_t rows_a = p.M - m0, rows_b = p.N - n0;
  const float* const A = static_cast<const float*>(p.A);
  const float* const B = static_cast<const float*>(p.B);
  const int64_t K1 = PH2 ? p.K1 : p.K;
  const int nk1 = static_cast<int>((K1 + kF32Step - 1) / kF32Step);
  const int nk = PH2 ? nk1 + static_cast<int>((p.K - K1 + kF32Step - 1) / kF32Step) : nk1;
  const int kv1 = static_cast<int>(K1 - static_cast<int64_t>(nk1 - 1) * kF32Step);
  const int kv2 = PH2 ? static_cast<int>(p.K - K1 - static_cast<int64_t>(nk - nk1 - 1) * kF32Step) : kv1;

  LA la, la2;
  LB lb;
  la.init(p.lda, rows_a, wave, lane);
  if constexpr (PH2) la2.init(p.lda2, rows_a, wave, lane);
  lb.init(p.ldb, rows_b, wave, lane);

  auto issue = [&](int kt) {
    char* st = smem + (kt % STAGES) * STAGE;
    const bool ph2 = PH2 && kt >= nk1;
    const int64_t k = static_cast<int64_t>(ph2 ? kt - nk1 : kt) * kF32Step;
    const int64_t kb = ph2 ? K1 + k : k;
    const int64_t lda = ph2 ? p.lda2 : p.lda;
    const float* a = ph2 ? static_cast<const float*>(p.A2) : A;
    a = AK ? a + m0 * lda + k : a + k * lda + m0;
    const float* b = BKM ? B + n0 * p.ldb + kb : B + kb * p.ldb + n0;
    const int kv = kt == nk - 1 ? kv2 : kt == nk1 - 1 ? kv1 : kF32Step;
    if (kv < kF32Step) {
      LA::load_tail(a, st, lda, rows_a, kv, wave, lane);
      LB::load_tail(b, st + A_BYTES, p.ldb, rows_b, kv, wave, lane);
    } else {
      if (ph2)
        la2.load(a, st, wave);
      else
        la.load(a, st, wave);
      lb.load(b, st + A_BYTES, wave);
    }
  };

  constexpr int ACC = f32_accs<TM, TN>();
  f32x16 accs[ACC][TM][TN];
#pragma unroll
  for (int q = 0; q < ACC; ++q)
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) accs[q][i][j][r] = 0.0f;
  float cs[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j) cs[j] = 0.0f;
  const bool do_colsum = EPI == EPI_DW && p.colsum != nullptr && tm == 0 && wm == 0;

  // The barrier of a k-tile stands before its last step: the next k-tile has
  // landed, every wave holds its last fragments, and the matrix cores work on
  // that step while the freed slot is refilled and the next k-tile's first
  // fragments are read.
  constexpr bool DW = EPI == EPI_DW;
  static_assert(kF32Step / 8 == 4, "four steps per k-tile");
  auto valid = [&](int kt) { return kt == nk - 1 ? kv2 : kt == nk1 - 1 ? kv1 : kF32Step; };
  auto zero_tail = [&](int kt) {
    if (valid(kt) < kF32Step) {
      char* st = smem + (kt % STAGES) * STAGE;
      f32_zero_tail<AK, BM, THREADS>(st, valid(kt), tid);
      f32_zero_tail<BKM, BN, THREADS>(st + A_BYTES, valid(kt), tid);
      __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): the LDS writes are done
      barrier_only();
    }
  };
#pragma unroll
  for (int s = 0; s < STAGES; ++s)
    if (s < nk) issue(s);
  wait_stage<LOADS, STAGES - 1>(nk < STAGES ? nk - 1 : STAGES - 1);
  barrier_only();
  zero_tail(0);
  const int arow = wm * (BM / WM), brow = wn * (BN / WN);
  float a[2][TM][4], b[2][TN][4];
#pragma unroll
  for (int i = 0; i < TM; ++i) f32_frag<AK, BM>(a[0][i], smem, arow + 32 * i, 0, lane);
#pragma unroll
  for (int j = 0; j < TN; ++j) f32_frag<BKM, BN>(b[0][j], smem + A_BYTES, brow + 32 * j, 0, lane);
  for (int kt = 0; kt < nk; ++kt) {
    const char* As = smem + (kt % STAGES) * STAGE;
    const char* Bs = As + A_BYTES;
    f32_step<AK, BKM, BM, BN, TM, TN, DW, 0>(a, b, As, Bs, 1, arow, brow, lane, accs, cs, do_colsum);
    f32_step<AK, BKM, BM, BN, TM, TN, DW, 1>(a, b, As, Bs, 2, arow, brow, lane, accs, cs, do_colsum);
    f32_step<AK, BKM, BM, BN, TM, TN, DW, 0>(a, b, As, Bs, 3, arow, brow, lane, accs, cs, do_colsum);
    __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): the last step's fragments
    const bool more = kt + 1 < nk;
    if (more) {
      const int left = nk - 2 - kt;
      wait_stage<LOADS, STAGES - 2>(left < STAGES - 2 ? left : STAGES - 2);
    }
    barrier_only();
    if (kt + STAGES < nk) issue(kt + STAGES);
    if (more) zero_tail(kt + 1);
    // (after the last k-tile these reads of another slot are not used)
    const char* An = smem + ((kt + 1) % STAGES) * STAGE;
    f32_step<AK, BKM, BM, BN, TM, TN, DW, 1>(a, b, An, An + A_BYTES, 0, arow, brow, lane, accs, cs,
                                             do_colsum);
  }

#pragma unroll
  for (int w = ACC / 2; w >= 1; w /= 2)
#pragma unroll
    for (int q = 0; q < w; ++q)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) accs[q][i][j] += accs[q + w][i][j];
  const f32x16 (&acc)[TM][TN] = accs[0];

  if constexpr (EPI == EPI_CHAIN) {
    // (one loss partial per wavefront, as the register-staged kernel's epilogue)
    float sq = 0.0f;
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int i = 0; i < TM; ++i)
        sq += chain_block(p, acc[i][j], m0 + wm * (BM / WM) + i * 32, n0 + wn * (BN / WN) + j * 32, lane);
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) sq += __shfl_xor(sq, o, 64);
    if (lane == 0) p.partials[static_cast<int64_t>(tile) * NW + wave] = sq;
    return;
  }
#pragma unroll
  for (int j = 0; j < TN; ++j)
#pragma unroll
    for (int i = 0; i < TM; ++i)
      store_block<float, float, EPI>(p, acc[i][j], m0 + wm * (BM / WM) + i * 32,
                                     n0 + wn * (BN / WN) + j * 32, lane);
  if constexpr (EPI == EPI_DW) {
    if (do_colsum) {
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const float t = cs[j] + __shfl_xor(cs[j], 32, 64);
        const int64_t col = n0 + wn * (BN / WN) + j * 32 + lane;
        if (lane < 32 && col < p.nvec) p.colsum[col] = t;
      }
    }
  }
}

template <bool AK, bool BKM, int BM, int BN, int WM, int WN, int STAGES, bool VEC, int EPI, bool PH2>
__global__ __launch_bounds__(64 * WM * WN, 2) void dlvm_gemm_f32_kernel(Params p) {
  __shared__ __attribute__((aligned(1024))) char smem[STAGES * (BM + BN) * kF32Step * 4];
  const int tile = split_slice<float, AK, BKM>(p, static_cast<int>(blockIdx.x));
  // (a k-slice of a split two-phase product lies in one phase)
  if (PH2 && p.splits <= 1)
    f32_gemm_tile<AK, BKM, BM, BN, WM, WN, STAGES, VEC, EPI, PH2>(p, tile, smem);
  else
    f32_gemm_tile<AK, BKM, BM, BN, WM, WN, STAGES, VEC, EPI, false>(p, tile, smem);
}

// The two adjoint products of one dense layer in one launch, as dlvm_gemm_pair_kernel.
template <int BM, int BN, int WM, int WN, int STAGES, bool VEC>
__global__ __launch_bounds__(64 * WM * WN, 2) void dlvm_gemm_f32_pair_kernel(Params p1, Params p2,
                                                                             int n1) {
  __shared__ __attribute__((aligned(1024))) char smem[STAGES * (BM + BN) * kF32Step * 4];
  const int b = static_cast<int>(blockIdx.x);
  if (b < n1) {
    const int tile = split_slice<float, false, false>(p1, b);
    f32_gemm_tile<false, false, BM, BN, WM, WN, STAGES, VEC, EPI_DW, false>(p1, tile, smem);
  } else {
    const int tile = split_slice<float, true, true>(p2, b - n1);
    f32_gemm_tile<true, true, BM, BN, WM, WN, STAGES, VEC, EPI_DACT, false>(p2, tile, smem);
  }
}

}  // namespace gemm
}  // namespace dlvm
