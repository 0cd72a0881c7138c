// The whole gradient of a small float32 softmax network in one workgroup.
//
// When the input, every weight and every layer output of a network fit in one
// compute unit's LDS and the products are tiny (the 64-32-10 network at batch
// 16 does 81K multiply-adds a step), a launch costs more than the work: the
// usual plan's launches are host-bound. Here one workgroup of 1024 threads
//   stages    the parameter block (every W_l and b_l, as it lies in memory),
//             x and the labels into LDS with plain contiguous copies (16-byte
//             loads where whole), all loads issued before the first store so
//             that HBM latency is paid once;
//   forward   H_{l+1} = act_l(H_l . W_l + b_l), the last layer giving logits;
//   loss      softmax cross-entropy (16 lanes per row up to 16 classes, else one
//             wave per row), and the adjoint of the logits (p - onehot) / B;
//   adjoint   per layer from the last: dW_l = H_l^T dZ, db_l = colsum dZ,
//             dZ_{l-1} = (dZ . W_l^T) * act'(H_l) (dx = dZ . W_0^T when x is
//             differentiated; the first layer's input adjoint is otherwise dead);
//   finalise  the mean loss, the device flags, the padding of dparams zeroed;
// with workgroup barriers between the phases and nothing but the results
// written to global memory. Every product runs on the matrix cores in 16 x 16 tiles
// (16x16x4 float32 instructions, operands read from LDS one value per lane and
// instruction), the tiles of a phase dealt to the waves; every sum runs in a fixed
// order, so the result is the same on every run.
//
// What bounds it is latency on one compute unit. With a thread per output the
// products were bound by LDS instructions (two reads per multiply-add; the 64-32-10
// network at batch 16 spent 5,560 cycles on its first forward product, 28,000 in all,
// 13.1 us a launch); a matrix instruction takes two reads for 1,024 multiply-adds. The
// kernel's arguments (1.2 KB; each 64-byte line a scalar load reaches for the first
// time takes 620 cycles, and the layer loops index them) are copied to LDS by one
// vector load beside the parameters; a phase's barrier waits for its LDS writes only,
// not for the gradients it stored; rows of at most 16 classes stay inside 16 lanes.
//
// LDS layout (words): the parameter block (W_l as [w_l][ldw_l], b_l, the
// padding between them); H_0 .. H_L as [B][hs_l]; two adjoint buffers
// [B][gs]; row losses, row label marks and labels [B] each. The row strides hs_l and
// gs are the widths rounded up to 4 more than a multiple of 8 where the budget allows
// (16 rows then lie in different banks), else the widths.
#include "common.hpp"
#include "kernels.hpp"

namespace dlvm {
namespace {

constexpr int kWaves = kSmallThreads / 64;
constexpr int kStage4 = kSmallMaxLds / 16 / kSmallThreads;  // 16-byte loads per thread and block

__device__ __forceinline__ float wave_sum(float v) {
  // butterfly: every lane ends with the same bits
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

__device__ __forceinline__ float wave_max(float v) {
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
  return v;
}

__device__ __forceinline__ int wave_or(int v) {
  for (int o = 32; o > 0; o >>= 1) v |= __shfl_xor(v, o);
  return v;
}

// One 16 x 16 tile of a product over K terms from LDS: A(m, k) at a[m * am + k * ak]
// for the tile's rows m < M (rows past it are read from row 0 and give outputs that
// are not stored), B(k, n) at b[n * bn + k * bk] for n < N. Lane 16 g + l of an
// instruction holds row (column) l at the g-th of its 4 k; the result's register r
// holds row 4 g + r, column l. Four accumulators take the instructions in turn:
// independent of each other, and shorter sums (outputs against float64 over 24 small
// networks: 1.11e-7 of the norm with two accumulators, 1.02e-7 with four, 1.06e-7 with
// lanes sharing a sum; 64-32-10 at batch 16 takes 7.7 us with two and 7.6 with four; over
// 250 networks of 8-128 inputs, batch 1-64, the four's errors are 0.93-0.98 of those of
// the shared sums in every gradient, though single networks go either way).
__device__ __forceinline__ f32x4 lds_tile(const float* __restrict__ a, int am, int ak, int M,
                                          const float* __restrict__ b, int bn, int bk, int N, int K,
                                          int lane) {
  const int l = lane & 15, g = lane >> 4;
  const float* pa = a + (l < M ? l * am : 0) + g * ak;
  const float* pb = b + (l < N ? l * bn : 0) + g * bk;
  f32x4 c[4] = {};
  const int full = K >> 2;
  int s = 0;
  for (; s + 4 <= full; s += 4) {
    float x[4], y[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      x[u] = pa[4 * u * ak];
      y[u] = pb[4 * u * bk];
    }
    pa += 16 * ak;
    pb += 16 * bk;
#pragma unroll
    for (int i = 0; i < 4; ++i) c[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[i], y[i], c[i], 0, 0, 0);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {  // at most 4 steps are left; the last one may hold fewer than 4 k
    if (4 * s >= K) break;
    const bool in = 4 * s + g < K;
    const float x = in ? *pa : 0.0f, y = in ? *pb : 0.0f;
    pa += 4 * ak;
    pb += 4 * bk;
    c[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(x, y, c[i], 0, 0, 0);
    ++s;
  }
  return (c[0] + c[1]) + (c[2] + c[3]);
}

// i / n for i < 2^16, n <= 2^12, with m = small_div(n).
__device__ __forceinline__ int div_by(int i, uint32_t m) {
  return m == 0u ? i : static_cast<int>(__umulhi(static_cast<uint32_t>(i), m));
}
__device__ __forceinline__ int tiles16(int n) { return (n + 15) >> 4; }

// The phases exchange through LDS: wait for this wave's LDS accesses, then for the
// other waves (global stores in flight are left alone; nothing here reads them back).
__device__ __forceinline__ void phase_barrier() {
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

struct SmallArgs {
  SmallNet t;
  const float* params;
  const float* x;
  const int32_t* labels;
  float* loss;
  float* dparams;
  float* dx;
  int32_t* flags;
  ZeroGaps gaps;
};
constexpr int kArgWords = sizeof(SmallArgs) / 4;
static_assert(sizeof(SmallArgs) % 4 == 0 && kArgWords <= kSmallThreads, "one word per thread");

__global__ __launch_bounds__(kSmallThreads) void dlvm_small_step_kernel(SmallArgs args) {
  __shared__ __attribute__((aligned(16))) float sm[kSmallLds / 4];
  __shared__ __attribute__((aligned(16))) uint32_t argw[kArgWords];
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, g16 = lane >> 4;
  // the arguments as words of the kernel-argument segment (its one argument is first)
  const uint32_t __attribute__((address_space(4)))* seg =
      (const uint32_t __attribute__((address_space(4)))*)__builtin_amdgcn_kernarg_segment_ptr();
  const uint32_t aw = tid < kArgWords ? seg[tid] : 0u;
  const SmallNet& t = reinterpret_cast<const SmallArgs*>(argw)->t;  // (after the first barrier)
  const ZeroGaps& gaps = reinterpret_cast<const SmallArgs*>(argw)->gaps;
  const float* __restrict__ params = args.params;
  const float* __restrict__ x = args.x;
  const int32_t* __restrict__ labels = args.labels;
  float* __restrict__ loss = args.loss;
  float* __restrict__ dparams = args.dparams;
  float* __restrict__ dx = args.dx;
  int32_t* __restrict__ flags = args.flags;
  const int B = args.t.B;

  // stage the parameter block, x and the labels (16-byte body, word tail)
  {
    const int pwords = args.t.pwords;
    const float* pb = params + args.t.pbase;
    const int w0 = args.t.w[0], xs_ld = args.t.hs[0];
    const uint32_t dx0 = args.t.divw0;
    const int np4 = pwords / 4, nx = B * w0, nx4 = nx / 4;
    float4 pv[kStage4], xv[kStage4];
#pragma unroll
    for (int j = 0; j < kStage4; ++j) {
      const int e = tid + j * kSmallThreads;
      if (e < np4) pv[j] = reinterpret_cast<const float4*>(pb)[e];
      if (e < nx4) xv[j] = reinterpret_cast<const float4*>(x)[e];
    }
    const int pt = np4 * 4 + tid, xt = nx4 * 4 + tid;
    const float ptail = pt < pwords ? pb[pt] : 0.0f;
    const float xtail = xt < nx ? x[xt] : 0.0f;
    const int lab = tid < B ? labels[tid] : 0;
    float* xs = sm + args.t.hoff[0];
    if (tid < kArgWords) argw[tid] = aw;
#pragma unroll
    for (int j = 0; j < kStage4; ++j) {
      const int e = tid + j * kSmallThreads;
      if (e < np4) reinterpret_cast<float4*>(sm)[e] = pv[j];
      if (e < nx4) {
        const float v[4] = {xv[j].x, xv[j].y, xv[j].z, xv[j].w};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int i = 4 * e + q, r = div_by(i, dx0);
          xs[r * xs_ld + i - r * w0] = v[q];
        }
      }
    }
    if (pt < pwords) sm[pt] = ptail;
    if (xt < nx) {
      const int r = div_by(xt, dx0);
      xs[r * xs_ld + xt - r * w0] = xtail;
    }
    if (tid < B) reinterpret_cast<int*>(sm + args.t.labels)[tid] = lab;
  }
  phase_barrier();

  // forward
  for (int l = 0; l < t.L; ++l) {
    const int K = t.w[l], N = t.w[l + 1], sw = t.ldw[l], act = t.act[l];
    const int hi = t.hs[l], ho = t.hs[l + 1];
    const float* h = sm + t.hoff[l];
    const float* W = sm + t.woff[l];
    const float* bias = sm + t.boff[l];
    float* o = sm + t.hoff[l + 1];
    const bool last = l == t.L - 1;
    const int tn = tiles16(N), nt = tiles16(B) * tn;
    for (int q = wave; q < nt; q += kWaves) {
      const int m0 = q / tn * 16, n0 = q % tn * 16;
      const f32x4 c = lds_tile(h + m0 * hi, hi, 1, B - m0, W + n0, 1, sw, N - n0, K, lane);
      const int n = n0 + l16;
      if (n < N) {
        const float bv = bias[n];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = m0 + 4 * g16 + r;
          const float v = c[r] + bv;
          if (row < B) o[row * ho + n] = last ? v : apply_act(act, v);
        }
      }
    }
    phase_barrier();
  }

  // softmax cross-entropy and the adjoint of the logits: at most 16 classes, one row
  // per 16 lanes; else one row per wave
  const int C = t.w[t.L], zs = t.hs[t.L], gs = t.gs;
  const float* Z = sm + t.hoff[t.L];
  float* rowloss = sm + t.rowloss;
  int* rowbad = reinterpret_cast<int*>(sm + t.rowbad);
  const int* lab = reinterpret_cast<const int*>(sm + t.labels);
  float* g = sm + t.g0;
  float* gn = sm + t.g1;
  if (C <= 16) {
    for (int r0 = wave * 4; r0 < B; r0 += kWaves * 4) {
      const int r = r0 + g16, rr = r < B ? r : 0;
      const float z = l16 < C ? Z[rr * zs + l16] : -INFINITY;
      const int y = lab[rr];
      const bool ok = y >= 0 && y < C;
      const float m = row16_max(z);
      const float e = l16 < C ? __expf(z - m) : 0.0f;
      const float s = row16_sum(e);
      if (r < B) {
        if (l16 == 0) {
          rowbad[r] = ok ? 0 : 1;
          rowloss[r] = ok ? (m + __logf(s)) - Z[r * zs + y] : NAN;
        }
        if (l16 < C) g[r * gs + l16] = t.scale / s * e - (l16 == y ? t.scale : 0.0f);
      }
    }
  } else {
    for (int r = wave; r < B; r += kWaves) {
      const float* z = Z + r * zs;
      float m = -INFINITY;
      for (int c = lane; c < C; c += 64) m = fmaxf(m, z[c]);
      m = wave_max(m);
      float s = 0.0f;
      for (int c = lane; c < C; c += 64) s += __expf(z[c] - m);
      s = wave_sum(s);
      const int y = lab[r];
      const bool ok = y >= 0 && y < C;
      if (lane == 0) {
        rowbad[r] = ok ? 0 : 1;
        rowloss[r] = ok ? (m + __logf(s)) - z[y] : NAN;
      }
      const float ps = t.scale / s;
      for (int c = lane; c < C; c += 64)
        g[r * gs + c] = ps * __expf(z[c] - m) - (c == y ? t.scale : 0.0f);
    }
  }
  phase_barrier();

  // the mean loss and the flags (the last wave, which gets the fewest tiles below;
  // nothing reads what it writes)
  if (wave == kWaves - 1) {
    float s = 0.0f;
    int bad = 0;
    for (int r = lane; r < B; r += 64) {
      s += rowloss[r];
      bad |= rowbad[r];
    }
    s = wave_sum(s);
    bad = wave_or(bad);
    if (lane == 0) {
      const float lv = s * t.scale;
      loss[0] = lv;
      flags[0] = bad ? 1 : 0;
      flags[1] = isfinite(lv) ? 0 : 1;
    }
  }

  // adjoint, last layer first: the tiles of dZ_{l-1} (or dx), then of dW, then the
  // column sums
  for (int l = t.L - 1; l >= 0; --l) {
    const int K = t.w[l], N = t.w[l + 1], ld = t.ldw[l], hi = t.hs[l];
    const float* W = sm + t.woff[l];
    const float* h = sm + t.hoff[l];
    float* dW = dparams + t.offW[l];
    float* db = dparams + t.offB[l];
    const int tk = tiles16(K), tl = tiles16(ld);
    const int nx = l > 0 || t.wrt_x ? tiles16(B) * tk : 0;
    const int nw = tk * tl, nb = tiles16(N);
    for (int q = wave; q < nx + nw + nb; q += kWaves) {
      if (q < nx) {
        const int m0 = q / tk * 16, k0 = q % tk * 16;
        const f32x4 c = lds_tile(g + m0 * gs, gs, 1, B - m0, W + k0 * ld, ld, 1, K - k0, N, lane);
        const int k = k0 + l16;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = m0 + 4 * g16 + r;
          if (k < K && row < B) {
            if (l > 0)
              gn[row * gs + k] = c[r] * act_grad_from_output(t.act[l - 1], h[row * hi + k]);
            else
              dx[row * K + k] = c[r];
          }
        }
      } else if (q < nx + nw) {
        // dW [K, ld] (padding columns zero)
        const int i = q - nx, k0 = i / tl * 16, n0 = i % tl * 16;
        const f32x4 c = lds_tile(h + k0, 1, hi, K - k0, g + n0, 1, gs, N - n0, B, lane);
        const int n = n0 + l16;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int k = k0 + 4 * g16 + r;
          if (k < K && n < ld) dW[k * ld + n] = n < N ? c[r] : 0.0f;
        }
      } else {
        // db [N]: 16 columns per wave, every fourth row per lane group
        const int n = (q - nx - nw) * 16 + l16;
        float s = 0.0f;
        if (n < N)
          for (int r = g16; r < B; r += 4) s += g[r * gs + n];
        s += __shfl_xor(s, 16, 64);
        s += __shfl_xor(s, 32, 64);
        if (g16 == 0 && n < N) db[n] = s;
      }
    }
    phase_barrier();
    float* tmp = g;
    g = gn;
    gn = tmp;
  }

  for (int q = wave; q < gaps.n; q += kWaves)
    for (int i = lane; i < gaps.len[q]; i += 64) dparams[gaps.off[q] + i] = 0.0f;
}

}  // namespace

// A factor m with __umulhi(i, m) == i / n for i < 2^16, 2 <= n <= 2^12:
// floor(2^32 / n) + 1 (its excess times i stays below 1 / n); 0 for n = 1.
static uint32_t small_div(int n) {
  return n == 1 ? 0u : static_cast<uint32_t>((uint64_t(1) << 32) / n + 1);
}

bool small_net(int L, const int32_t* widths, const int32_t* acts, const int64_t* offsets,
               const int64_t* ldw, int64_t B, bool wrt_x, SmallNet& t) {
  if (L < 1 || L > kSmallMaxLayers || B < 1 || B > 1024) return false;
  t = SmallNet{};
  t.L = L;
  t.B = static_cast<int>(B);
  t.wrt_x = wrt_x ? 1 : 0;
  for (int l = 0; l <= L; ++l) {
    if (widths[l] < 1 || widths[l] > 4096) return false;
    t.w[l] = widths[l];
    t.maxw = widths[l] > t.maxw ? widths[l] : t.maxw;
  }
  // LDS layout, in words, checked against the budget before any narrowing;
  // blocks start on 4-word (16-byte) boundaries
  const int64_t pbase = offsets[0];
  const int64_t pwords = offsets[2 * L - 1] + widths[L] - pbase;
  int64_t words = 0;
  auto take = [&](int64_t n) {
    const int64_t o = words;
    words += (n + 3) / 4 * 4;
    return o;
  };
  take(pwords);
  int64_t hoff[kSmallMaxLayers + 1];
  for (int l = 0; l <= L; ++l) hoff[l] = take(B * widths[l]);
  int64_t g0 = take(B * t.maxw), g1 = take(B * t.maxw);
  int64_t rl = take(B), rb = take(B), lb = take(B);
  int64_t macs = 0;
  for (int l = 0; l < L; ++l) {
    if (ldw[l] > 4096) return false;
    macs += 3 * B * int64_t(widths[l]) * widths[l + 1];
  }
  if (words > kSmallMaxLds / 4 || macs > kSmallMaxMacs) return false;
  // the rows apart (see the layout above) where that fits the workgroup's LDS
  auto apart = [](int w) { return (w + 3) / 8 * 8 + 4; };
  static_assert(kSmallLds >= kSmallMaxLds, "unpadded rows always fit");
  for (int pad = 1; pad >= 0; --pad) {
    t.gs = pad ? apart(t.maxw) : t.maxw;
    words = 0;
    take(pwords);
    for (int l = 0; l <= L; ++l) {
      t.hs[l] = pad ? apart(widths[l]) : widths[l];
      hoff[l] = take(B * t.hs[l]);
    }
    g0 = take(B * t.gs);
    g1 = take(B * t.gs);
    rl = take(B);
    rb = take(B);
    lb = take(B);
    if (words <= kSmallLds / 4) break;
  }
  t.pbase = pbase;
  t.pwords = static_cast<int>(pwords);
  for (int l = 0; l <= L; ++l) t.hoff[l] = static_cast<int>(hoff[l]);
  t.g0 = static_cast<int>(g0);
  t.g1 = static_cast<int>(g1);
  t.rowloss = static_cast<int>(rl);
  t.rowbad = static_cast<int>(rb);
  t.labels = static_cast<int>(lb);
  for (int l = 0; l < L; ++l) {
    t.act[l] = acts[l];
    t.woff[l] = static_cast<int>(offsets[2 * l] - pbase);
    t.boff[l] = static_cast<int>(offsets[2 * l + 1] - pbase);
    t.offW[l] = offsets[2 * l];
    t.offB[l] = offsets[2 * l + 1];
    t.ldw[l] = static_cast<int>(ldw[l]);
  }
  t.divw0 = small_div(widths[0]);
  t.scale = static_cast<float>(1.0 / static_cast<double>(B));
  return true;
}

hipError_t launch_small_step(const SmallNet& t, const float* params, const float* x,
                             const int32_t* labels, float* loss, float* dparams, float* dx,
                             int32_t* flags, const ZeroGaps& gaps, hipStream_t s) {
  if (t.pwords > kSmallMaxLds / 4 || t.B * t.w[0] > kSmallMaxLds / 4) return hipErrorInvalidValue;
  const SmallArgs a{t, params, x, labels, loss, dparams, dx, flags, gaps};
  launch_kernel(dlvm_small_step_kernel, dim3(1), dim3(kSmallThreads), s, a);
  return hipGetLastError();
}

}  // namespace dlvm
