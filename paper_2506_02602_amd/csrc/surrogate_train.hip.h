// Training step of the surrogate MLP in two kernels per batch (BF16 MFMA,
// FP32 accumulation; the BF16 rounding points are those of the forward and
// backward passes the oracle emulates):
//
//   train_fb   one block per 16 samples, one wave per 16 of the 128 hidden
//              features: gather the batch rows through the epoch's
//              permutation, the forward pass, the loss and its gradient, and
//              back through the layers, dZ_l = BF16(dH_l * silu'(Z_l)), with
//              the pre-activations in registers; the waves exchange each
//              layer's BF16 activations (then gradients) through LDS.  It
//              leaves what the weight gradients need, feature-major (one row
//              of samples per feature): inputs, H_l, dZ_l and the output
//              gradient;
//   train_dw   one block per 16 x 16 tile of a weight gradient: the
//              batch's dZ_l^T H_(l-1) as MFMA chains over the samples, split
//              over the block's waves and added in wave order (both operands
//              sample-contiguous rows), the bias gradient from
//              the same dZ rows, then either the gradient itself or the Adam
//              update of those parameters, written to the FP32 masters, the
//              BF16 natural copy and both packed layouts (no reduction or
//              repacking pass).
#pragma once

namespace surr {

// inverse of packed_feature: the packed column of hidden feature f
__host__ __device__ constexpr int packed_column(int f) {
  return (f & ~31) + (((f & 31) < 16) ? 8 * ((f & 15) >> 2) + (f & 3)
                                      : 8 * ((f & 15) >> 2) + 4 + (f & 3));
}

constexpr bool packed_column_inverts() {
  for (int c = 0; c < HID; ++c)
    if (packed_column(packed_feature(c)) != c) return false;
  return true;
}
static_assert(packed_column_inverts(), "packed_column is the inverse of packed_feature");

struct TrainArgs {
  // batch rows: sample s of the batch is row (pa ((first + s) mod n) + pb) mod n
  const float* Xn; const float* Yn; long n; long first; unsigned long long pa, pb;
  int B, Bp;                         // batch size, and rounded up to 32 (row stride)
  const unsigned short* wpack; const float* bpack;   // forward (inference) layout
  const unsigned short* wtpack;                      // transposed layout for dH = W^T dZ
  unsigned short* Xfm;               // [NI16][Bp] BF16 inputs, feature-major
  unsigned short* Hfm;               // [3][HID][Bp] BF16 activations
  unsigned short* dZfm;              // [3][HID][Bp] BF16 pre-activation gradients
  unsigned short* doutfm;            // [NO16][Bp] BF16 output gradient
  double* sse; float scale;          // sum of squared errors; 2 / (B NO)
  // train_dw
  float* theta; float* m; float* v; float* grad; unsigned short* wbf;
  unsigned short* wpack_w; float* bpack_w; unsigned short* wtpack_w;
  int adam; float lr, b1, b2, c1, c2, eps;
  long oW[4], ob[4];
};

template <class M>
struct TrainShape {
  using S = InferShape<M>;
  static constexpr int NI = S::NI, NO = S::NO, KC1 = S::KC1, OT4 = S::OT4;
  static constexpr int NI16 = (NI + 15) / 16 * 16, NO16 = OT4 * 16;
  static constexpr int KO = (NO + 31) / 32;            // k chunks of dH_3 = W4^T dout
  static constexpr int W4T_LD = KO * 32 + kRowPad;
  static constexpr long WT4 = (long)HID * W4T_LD, WT2 = (long)HID * kWLd;
  static constexpr long WTTOT = WT4 + 2 * WT2;         // [W4^T][W3^T][W2^T]
  // train_fb: TS samples per block, one wave per 16 hidden features
  static constexpr int TS = 16, WAVES = HID / 16;
  static_assert(OT4 <= WAVES, "one output tile per wave");
  // train_dw work items: (layer, out tile, in tile)
  static constexpr int IT1 = NI16 / 16, OTH = HID / 16, ITH = HID / 16;
  static constexpr int N1 = OTH * IT1, N2 = OTH * ITH, N4 = OT4 * ITH;
  static constexpr int ITEMS = N1 + 2 * N2 + N4;
};

__device__ __forceinline__ float dsilu_fast(float z) {
  const float s = __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * z));
  return s * (1.0f + z * (1.0f - s));
}

// x mod n for x <= n^2 (a permutation's multiplier and offset are below n, a
// batch ends before the second epoch): for n below 2^31 from the FP64 quotient,
// which is below 2^31 then and off by at most one, in place of a 64-bit
// division.
__device__ __forceinline__ unsigned long long mod_n(unsigned long long x, unsigned long long n) {
  if (x < n) return x;
  if (n >= (1ull << 31) || x >= (1ull << 62)) return x % n;
  const unsigned long long q = (unsigned long long)((double)x * (1.0 / (double)n));
  long long r = (long long)(x - q * n);
  if (r < 0) r += (long long)n;
  if (r >= (long long)n) r -= (long long)n;
  return (unsigned long long)r;
}

__device__ __forceinline__ long batch_row(const TrainArgs& a, int s) {
  const unsigned long long n = (unsigned long long)a.n;
  return (long)mod_n(a.pa * mod_n((unsigned long long)(a.first + s), n) + a.pb, n);
}

// What bounds it: latency, a chain of seven small products with an exchange
// between each.  A wave that took all 128 features of its 16 samples left three
// quarters of the chip idle and did 76 MFMAs and 32 activations per layer in
// sequence (forward and backward 31.4 us for 4,096 samples, in two kernels that
// passed the pre-activations through memory); split over 8 waves the same
// products, in the same order of accumulation, are 19 to 23 MFMAs per wave on
// every CU (11.8 us).  The wave's weights come straight from the packed panels (L2) into
// registers, loaded before they are needed.
template <class M>
__global__ __launch_bounds__(64 * TrainShape<M>::WAVES) void train_fb(TrainArgs a) {
  using T = TrainShape<M>;
  using S = typename T::S;
  constexpr int NI = T::NI, NO = T::NO, KC1 = T::KC1, OT4 = T::OT4, KO = T::KO;
  constexpr int XLD = KC1 * 32 + kRowPad, OLD = KO * 32 + kRowPad;
  __shared__ __attribute__((aligned(16))) unsigned short sX[T::TS][XLD];
  __shared__ __attribute__((aligned(16))) unsigned short sH[2][T::TS][kWLd];
  __shared__ __attribute__((aligned(16))) unsigned short sO[T::TS][OLD];
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int g = lane >> 4, r16 = lane & 15;
  const int s = blockIdx.x * T::TS + r16;      // this lane's sample
  const bool in = s < a.B;
  const long row = in ? batch_row(a, s) : 0;
  const int feat = 16 * wave + 4 * g;          // this lane's first hidden feature
  // this lane's inputs and targets
  float xv[KC1], yv[4];
#pragma unroll
  for (int kc = 0; kc < KC1; ++kc) {
    const int k = kc * 32 + 4 * wave + g;
    xv[kc] = in && k < NI ? a.Xn[row * NI + k] : 0.f;
  }
#pragma unroll
  for (int i = 0; i < 4; ++i)
    yv[i] = wave < OT4 && in && feat + i < NO ? a.Yn[row * NO + feat + i] : 0.f;
  // this wave's rows of the weights (A operands) and its biases
  const unsigned short* wp = a.wpack + (long)(16 * wave + r16) * S::W1_LD + 8 * g;
  const unsigned short* w2 = a.wpack + S::W1 + (long)(16 * wave + r16) * kWLd + 8 * g;
  v8s w1[KC1], wf[2][4];
#pragma unroll
  for (int kc = 0; kc < KC1; ++kc) w1[kc] = *reinterpret_cast<const v8s*>(wp + kc * 32);
#pragma unroll
  for (int l = 0; l < 2; ++l)
#pragma unroll
    for (int kc = 0; kc < 4; ++kc) wf[l][kc] = *reinterpret_cast<const v8s*>(w2 + l * S::W2 + kc * 32);
  f32x4 bias[3], bias4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int l = 0; l < 3; ++l) bias[l] = *reinterpret_cast<const f32x4*>(a.bpack + l * HID + feat);
  v8s w4[4] = {};
  if (wave < OT4) {
    const unsigned short* q = a.wpack + S::W1 + 2 * S::W2 + (long)(16 * wave + r16) * kWLd + 8 * g;
#pragma unroll
    for (int kc = 0; kc < 4; ++kc) w4[kc] = *reinterpret_cast<const v8s*>(q + kc * 32);
    bias4 = *reinterpret_cast<const f32x4*>(a.bpack + 3 * HID + feat);
  }
#pragma unroll
  for (int kc = 0; kc < KC1; ++kc) {
    const int k = kc * 32 + 4 * wave + g;
    const unsigned short x = f2bf(xv[kc]);
    sX[r16][k] = x;
    if (k < T::NI16) a.Xfm[(long)k * a.Bp + s] = x;
  }
  // the output gradient's columns past the output tiles
  for (int k = OT4 * 16 + (tid >> 4); k < KO * 32; k += 4 * T::WAVES) sO[tid & 15][k] = 0;
  __syncthreads();
  f32x4 acc = bias[0];
#pragma unroll
  for (int kc = 0; kc < KC1; ++kc)
    acc = mfma(w1[kc], *reinterpret_cast<const v8s*>(&sX[r16][kc * 32 + 8 * g]), acc);
  // this lane's four features in the packed column order of the next layer
  const int pcol = 32 * (wave >> 1) + 8 * g + 4 * (wave & 1);
  f32x4 z[3];
#pragma unroll
  for (int l = 0; l < 3; ++l) {
    z[l] = acc;
    unsigned short h[4];
    unsigned short* hl = a.Hfm + ((long)l * HID + feat) * a.Bp + s;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      h[i] = in ? f2bf(silu_fast(acc[i])) : (unsigned short)0;
      hl[(long)i * a.Bp] = h[i];
    }
    *reinterpret_cast<ushort4*>(&sH[l & 1][r16][pcol]) = ushort4{h[0], h[1], h[2], h[3]};
    __syncthreads();
    if (l == 2) break;
    acc = bias[l + 1];
#pragma unroll
    for (int kc = 0; kc < 4; ++kc)
      acc = mfma(wf[l][kc], *reinterpret_cast<const v8s*>(&sH[l & 1][r16][kc * 32 + 8 * g]), acc);
  }
  // the transposed weights for the way back
  const unsigned short* wt = a.wtpack + (long)(16 * wave + r16) * T::W4T_LD + 8 * g;
  const unsigned short* wt3 = a.wtpack + T::WT4 + (long)(16 * wave + r16) * kWLd + 8 * g;
  v8s wt4[KO], wb[2][4];
#pragma unroll
  for (int kc = 0; kc < KO; ++kc) wt4[kc] = *reinterpret_cast<const v8s*>(wt + kc * 32);
#pragma unroll
  for (int l = 0; l < 2; ++l)
#pragma unroll
    for (int kc = 0; kc < 4; ++kc) wb[l][kc] = *reinterpret_cast<const v8s*>(wt3 + l * T::WT2 + kc * 32);
  // ---- outputs, loss and its gradient dL/dout = 2 (out - y) / (B NO), BF16
  if (wave < OT4) {
    acc = bias4;
#pragma unroll
    for (int kc = 0; kc < 4; ++kc)
      acc = mfma(w4[kc], *reinterpret_cast<const v8s*>(&sH[0][r16][kc * 32 + 8 * g]), acc);
    double se = 0.0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      unsigned short d16 = 0;
      if (feat + i < NO && in) {
        const float d = acc[i] - yv[i];
        d16 = f2bf(a.scale * d);
        se += (double)d * d;
      }
      sO[r16][feat + i] = d16;
      a.doutfm[(long)(feat + i) * a.Bp + s] = d16;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) se += __shfl_xor(se, off);
    if (lane == 0) atomicAdd(a.sse, se);
  }
  __syncthreads();
  // ---- back: dH_3 = W4^T dout, dZ_l = BF16(dH_l * silu'(Z_l)), dH_(l-1) = W_l^T dZ_l
  acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int kc = 0; kc < KO; ++kc)
    acc = mfma(wt4[kc], *reinterpret_cast<const v8s*>(&sO[r16][kc * 32 + 8 * g]), acc);
#pragma unroll
  for (int l = 2; l >= 0; --l) {
    unsigned short d[4];
    unsigned short* dl = a.dZfm + ((long)l * HID + feat) * a.Bp + s;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      d[i] = in ? f2bf(acc[i] * dsilu_fast(z[l][i])) : (unsigned short)0;
      dl[(long)i * a.Bp] = d[i];
    }
    if (l == 0) break;
    *reinterpret_cast<ushort4*>(&sH[(l + 1) & 1][r16][pcol]) = ushort4{d[0], d[1], d[2], d[3]};
    __syncthreads();
    acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kc = 0; kc < 4; ++kc)
      acc = mfma(wb[2 - l][kc], *reinterpret_cast<const v8s*>(&sH[(l + 1) & 1][r16][kc * 32 + 8 * g]),
                 acc);
  }
}

// One FP32 master parameter with its moments.
struct AdamState { float th, m, v; };

// Adam on it (the moment decay rates and the bias corrections as FP32
// numbers); returns the new value
__device__ __forceinline__ float adam_one(const TrainArgs& a, long p, const AdamState& o, float gr) {
  const float mi = a.b1 * o.m + (1.f - a.b1) * gr;
  const float vi = a.b2 * o.v + (1.f - a.b2) * gr * gr;
  a.m[p] = mi;
  a.v[p] = vi;
  const float th = o.th - a.lr * (mi / a.c1) / (sqrtf(vi / a.c2) + a.eps);
  a.theta[p] = th;
  return th;
}

constexpr int kDwWaves = 16;

template <class M>
__global__ __launch_bounds__(64 * kDwWaves) void train_dw(TrainArgs a) {
  using T = TrainShape<M>;
  using S = typename T::S;
  constexpr int NI = T::NI, NO = T::NO;
  __shared__ float red[kDwWaves][5][64];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, g = lane >> 4, r16 = lane & 15;
  // one block per item: layer l (0-based: W1..W4), out tile ot, in tile it
  int item = blockIdx.x;
  int l, ot, it;
  if (item < T::N1) { l = 0; ot = item / T::IT1; it = item % T::IT1; }
  else if ((item -= T::N1) < 2 * T::N2) { l = 1 + item / T::N2; item %= T::N2; ot = item / T::ITH; it = item % T::ITH; }
  else { item -= 2 * T::N2; l = 3; ot = item / T::ITH; it = item % T::ITH; }
  const int out_dim = l == 3 ? NO : HID, in_dim = l == 0 ? NI : HID;
  const unsigned short* A = l == 3 ? a.doutfm : a.dZfm + (long)l * HID * a.Bp;     // [out][Bp]
  const unsigned short* Bm = l == 0 ? a.Xfm : a.Hfm + (long)(l - 1) * HID * a.Bp;  // [in][Bp]
  const unsigned short* arow = A + (long)(ot * 16 + r16) * a.Bp + 8 * g;
  const unsigned short* brow = Bm + (long)(it * 16 + r16) * a.Bp + 8 * g;
  // the waves split the samples; each sums its share, the first wave adds
  // the shares in wave order
  const int per = (a.Bp / 32 + kDwWaves - 1) / kDwWaves * 32;
  const int kb = wave * per, ke = min(kb + per, a.Bp);
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  float bsum = 0.f;
  const bool bias_tile = it == 0;
  // After the split sums, wave i < 4 takes parameter D[4g + i][r16] = dW[out =
  // 16 ot + 4g + i][in = 16 it + r16] of its lanes and wave 4 the biases: the
  // masters and moments are loaded now, under the products.  (11.0 us per batch
  // of 4,096; one wave doing all of it after the sums: 13.5.)
  const int o = wave == 4 ? ot * 16 + r16 : ot * 16 + 4 * g + wave, inp = it * 16 + r16;
  const bool mine = wave < 4 ? o < out_dim && inp < in_dim
                             : wave == 4 && bias_tile && g == 0 && o < out_dim;
  const long p = wave < 4 ? a.oW[l] + (long)o * in_dim + inp : a.ob[l] + o;
  AdamState st{0.f, 0.f, 0.f};
  if (mine && a.adam) st = AdamState{a.theta[p], a.m[p], a.v[p]};
#pragma unroll 8
  for (int k0 = kb; k0 < ke; k0 += 32) {
    const v8s av = *reinterpret_cast<const v8s*>(arow + k0);
    const v8s bv = *reinterpret_cast<const v8s*>(brow + k0);
    acc = mfma(av, bv, acc);
    if (bias_tile) {
#pragma unroll
      for (int j = 0; j < 8; ++j) bsum += bf2f((unsigned short)av[j]);
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) red[wave][i][lane] = acc[i];
  red[wave][4][lane] = bsum;
  __syncthreads();
  if (wave > 4 || (wave == 4 && !bias_tile)) return;
  // the waves' shares in wave order
  float sum = red[0][wave][lane];
#pragma unroll
  for (int w = 1; w < kDwWaves; ++w) sum += red[w][wave][lane];
  if (wave == 4) {
    // the four lanes of one out row (g = 0..3) hold its partial sums
    sum += __shfl_xor(sum, 16);
    sum += __shfl_xor(sum, 32);
  }
  if (!mine) return;
  if (!a.adam) { a.grad[p] = sum; return; }
  const float th = adam_one(a, p, st, sum);
  const unsigned short b16 = f2bf(th);
  a.wbf[p] = b16;
  if (wave == 4) {
    a.bpack_w[l * HID + o] = th;
  } else if (l == 0) {
    // the forward (inference) layout and the transposed backward one
    a.wpack_w[(long)o * S::W1_LD + inp] = b16;
  } else {
    a.wpack_w[S::W1 + (long)(l - 1) * S::W2 + (long)o * kWLd + packed_column(inp)] = b16;
    if (l == 3) a.wtpack_w[(long)inp * T::W4T_LD + o] = b16;
    else a.wtpack_w[T::WT4 + (long)(2 - l) * T::WT2 + (long)inp * kWLd + packed_column(o)] = b16;
  }
}

// theta -> the transposed backward layout (initial packing; the training
// step keeps it current for the parameters it updates)
__global__ void pack_transposed(const float* theta, int ni, int no, long oW2, long oW3, long oW4,
                                int w4t_ld, long wt4, long wt2, unsigned short* wt) {
  const long total = wt4 + 2 * wt2;
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < total;
       i += (long)gridDim.x * blockDim.x) {
    unsigned short v = 0;
    if (i < wt4) {
      const long in = i / w4t_ld, o = i % w4t_ld;
      if (o < no) v = f2bf(theta[oW4 + o * HID + in]);
    } else {
      const long j = i - wt4, which = j / wt2, jj = j % wt2, in = jj / kWLd, c = jj % kWLd;
      const long base = which == 0 ? oW3 : oW2;
      if (c < HID) v = f2bf(theta[base + (long)packed_feature((int)c) * HID + in]);
    }
    wt[i] = v;
  }
}

}  // namespace surr

template <class M>
hipError_t launch_train(const surr::TrainArgs& a, int phase, hipStream_t s) {
  using T = surr::TrainShape<M>;
  if (phase == 0)
    hipLaunchKernelGGL(surr::train_fb<M>, dim3((unsigned)(a.Bp / T::TS)), dim3(64 * T::WAVES), 0, s,
                       a);
  else
    hipLaunchKernelGGL(surr::train_dw<M>, dim3(T::ITEMS), dim3(64 * surr::kDwWaves), 0, s, a);
  return hipGetLastError();
}

template <class M>
struct TrainSizes {
  using T = surr::TrainShape<M>;
  static constexpr long wtpack_elems = T::WTTOT;
  static constexpr int ni16 = T::NI16, no16 = T::NO16, w4t_ld = T::W4T_LD;
  static constexpr long wt4 = T::WT4, wt2 = T::WT2;
};
