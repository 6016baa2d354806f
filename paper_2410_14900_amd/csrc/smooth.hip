// Gaussian smoothing of the learned redundancy weight (paper Sec. 3.1: a Gaussian
// filter layer after the weight layer) and its exact transpose.
//
//   Ms = G_mu G_s M   per view,   (G x)[i] = sum_{t=-r..r} w_t x[mirror(i + t)],
//   w_t = exp(-t^2 / (2 sigma^2)) normalised over t = -r..r,
//   mirror(m) = -m (m < 0), m, 2(n-1) - m (m > n-1)   (edge sample not repeated).
//
// Each 1D pass stages whole lines in LDS with r-sample halos, zero-padded to a pitch of P
// samples; a thread forms kOB consecutive outputs of a line from a window of 16 samples in
// registers, which one 16-byte LDS read moves by four taps (48 FMAs).  The forward pass fills
// the halos by mirroring.  The transpose of one pass is
//   gx[j] = C(j) + [j > 0] C(-j) + [j < n-1] C(2(n-1) - j),
//   C(c)  = sum_t w_t gy[c - t]  over 0 <= c - t < n,
// i.e. the same convolution with zero halos (the symmetric w makes it a correlation), also
// at the r positions beyond each end, whose values the outputs at their mirror images
// receive.  Blocks beyond the ends skip the taps that only meet zeros (half of them).  Every
// workgroup reads all it writes before its barrier and workgroups touch disjoint lines, so
// both passes may run in place.
//
// Bound by the FMAs: 2 r + 1 per output and pass.  kOB = 12 keeps the LDS reads of
// neighbouring blocks of a line (12 samples apart) and of neighbouring lines (P = 4 mod 32)
// free of bank conflicts.  248 views of 360 x 725 at r = 60, forward and transpose: 2.80 ms with
// four outputs per thread, whose window moved one sample per read, 1.08 ms so (half of it the
// FMAs at the rate the vector units reach; 0.36 ms its memory traffic at a copy's rate).
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "dc_internal.h"

namespace dc {

typedef float f32x4 __attribute__((ext_vector_type(4)));

static constexpr int kOB = 12;        // consecutive outputs per thread
static constexpr int kSmCols = 16;    // s-columns in the mu pass's LDS limit
static constexpr int kFront = 16;     // zeros before a line's halo in the transpose, which rounds taps down to fours

static __host__ __device__ int blocks_of(int n) { return (n + kOB - 1) / kOB; }
// blocks of a line before, in and after it (the transpose's outputs reach r beyond the ends)
struct LineBlocks {
  int left, mid, right;
  __host__ __device__ LineBlocks(bool adj, int n, int r)
      : left(adj ? blocks_of(r) : 0), mid(blocks_of(n)), right(adj ? blocks_of(max2(n + r - kOB * mid)) : 0) {}
  __host__ __device__ int all() const { return left + mid + right; }
  static __host__ __device__ int max2(int x) { return x > 0 ? x : 0; }
};
// samples per staged line: its blocks, the halos and 4 read past them; 4 mod 32
static __host__ __device__ int line_pitch(bool adj, int n, int r) {
  const LineBlocks b(adj, n, r);
  return ((adj ? kFront : 0) + kOB * (b.all() - b.left) + 2 * r + 4 + 27) / 32 * 32 + 4;
}
static __host__ __device__ int tap_words(int r) { return (2 * r + 1 + 3) / 4 * 4; }

// acc[k] += w[u] v[u + k], u = 0..3, over the window v = a, b, c, d
template <int TAPS>
__device__ __forceinline__ void taps(f32x4 w, f32x4 a, f32x4 b, f32x4 c, f32x4 d, float (&acc)[kOB]) {
  const float v[16] = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3], c[0], c[1], c[2], c[3], d[0], d[1], d[2], d[3]};
#pragma unroll
  for (int u = 0; u < TAPS; ++u)
#pragma unroll
    for (int k = 0; k < kOB; ++k) acc[k] = fmaf(w[u], v[u + k], acc[k]);
}

// kOB outputs sum_t w[t] line[t + k], t = t0..t1-1 in order; t0 a multiple of 4 and
// t1 - t0 odd or a multiple of 4
__device__ __forceinline__ void conv_run(const float* __restrict__ line, const float* __restrict__ w, int t0, int t1,
                                         float (&acc)[kOB]) {
  const f32x4* v = reinterpret_cast<const f32x4*>(line + t0);
  const f32x4* wv = reinterpret_cast<const f32x4*>(w + t0);
  f32x4 a = v[0], b = v[1], c = v[2], d;
#pragma unroll
  for (int k = 0; k < kOB; ++k) acc[k] = 0.f;
  int t = t0;
  for (; t + 16 <= t1; t += 16) {
    v += 4;
    d = v[-1];
    taps<4>(wv[0], a, b, c, d, acc);
    a = v[0];
    taps<4>(wv[1], b, c, d, a, acc);
    b = v[1];
    taps<4>(wv[2], c, d, a, b, acc);
    c = v[2];
    taps<4>(wv[3], d, a, b, c, acc);
    wv += 4;
  }
  for (; t + 4 <= t1; t += 4) {
    ++v;
    d = v[2];
    taps<4>(*wv++, a, b, c, d, acc);
    a = b;
    b = c;
    c = d;
  }
  if (t + 1 == t1) taps<1>(*wv, a, b, c, d, acc);
  if (t + 3 == t1) taps<3>(*wv, a, b, c, v[3], acc);
}

// One workgroup: `lines` lines of n samples.  The s-pass (MU false) takes consecutive rows of
// the sinograms; the mu-pass takes columns, neighbouring ones in neighbouring lanes, and all
// of a view's on one XCD, whose L2 then holds the memory lines that two workgroups share.
// The forward mu-pass stores its outputs as it forms them (a row of `lines` values at a
// time) and may take its items in several rounds; the others hold them in registers, at most
// ROUNDS items per thread, and leave through LDS, for contiguous stores and, in the
// transpose, the mirrored sums.
// lds = taps [2r + 1, padded to 4], lines [lines][pitch]
template <bool ADJ, bool MU, int ROUNDS>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(ROUNDS == 1 ? 8 : 6))) void k_smooth(const float* in, float* out, int n_theta, int ns, GaussTaps tp,
                                                 int r, int v0, int nv, int lines, int strips) {
  constexpr bool STAGED = ADJ || !MU;
  extern __shared__ float sm[];
  const int n = MU ? n_theta : ns, pitch = line_pitch(ADJ, n, r);
  constexpr int front = ADJ ? kFront : 0;
  const LineBlocks lb(ADJ, n, r);
  float* w = sm;
  float* buf = w + tap_words(r);
  size_t base;
  int held;   // lines of this workgroup
  if (MU) {
    const int kb = blockIdx.x >> 3, vl = (blockIdx.x & 7) + 8 * (kb / strips), c0 = kb % strips * lines;
    if (vl >= nv) return;
    base = (size_t)(v0 + vl) * n_theta * ns + c0;
    held = min(lines, ns - c0);
  } else {
    const size_t l0 = (size_t)blockIdx.x * lines;
    base = ((size_t)v0 * n_theta + l0) * ns;
    held = (int)min((size_t)lines, (size_t)nv * n_theta - l0);
  }
  const int sh = 31 - __clz(lines);   // MU: lines is a power of two
  for (int q = threadIdx.x; q < tap_words(r); q += blockDim.x) w[q] = q > 2 * r ? 0.f : tp.w[q < r ? r - q : q - r];
  auto source = [&](int m) {   // the sample at position m, -1 for a zero
    if (m >= 0 && m < n) return m;
    if (ADJ || m < -r || m > n - 1 + r) return -1;
    return m < 0 ? -m : 2 * (n - 1) - m;
  };
  // kLoad samples in flight per thread
  constexpr int kLoad = 8;
  const int total = MU ? pitch << sh : held * pitch;
  int l = 0, m = threadIdx.x;   // S: line and sample of the thread's next word
  for (int q0 = threadIdx.x; q0 < total; q0 += kLoad * blockDim.x) {
    float x[kLoad];
    int at[kLoad];
#pragma unroll
    for (int u = 0; u < kLoad; ++u) {
      const int q = q0 + u * blockDim.x;
      int src;
      if (MU) {
        l = q & (lines - 1);
        m = q >> sh;
      } else {
        while (m >= pitch) {
          m -= pitch;
          ++l;
        }
      }
      src = source(m - r - front);
      at[u] = l * pitch + m;
      x[u] = q < total && src >= 0 && l < held ? in[base + (MU ? (size_t)src * ns + l : (size_t)l * ns + src)] : 0.f;
      if (!MU) m += blockDim.x;
    }
#pragma unroll
    for (int u = 0; u < kLoad; ++u)
      if (q0 + u * blockDim.x < total) buf[at[u]] = x[u];
  }
  __syncthreads();
  // an item is a line and a block of it, c0 = 12 block its first position; blocks beyond the
  // ends come last
  const int items = held * lb.all();
  auto place = [&](int q, int& l, int& c0) {
    const int mids = held * lb.mid, e = q < mids ? q : q - mids, nb = q < mids ? lb.mid : lb.all() - lb.mid;
    int b;
    if (MU) {
      b = e / held;
      l = e - b * held;
    } else {
      l = e / nb;
      b = e - l * nb;
    }
    if (q >= mids) b = b < lb.left ? b - lb.left : lb.mid + b - lb.left;
    c0 = b * kOB;
  };
  if (!STAGED) {
    for (int q = threadIdx.x; q < items; q += blockDim.x) {
      int l, c0;
      place(q, l, c0);
      float acc[kOB];
      conv_run(buf + l * pitch + c0, w, 0, 2 * r + 1, acc);
#pragma unroll
      for (int k = 0; k < kOB; ++k)
        if (c0 + k < n) out[base + (size_t)(c0 + k) * ns + l] = acc[k];
    }
    return;
  }
  float acc[ROUNDS][kOB];
#pragma unroll
  for (int p = 0; p < ROUNDS; ++p) {
    const int q = p * blockDim.x + threadIdx.x;
    if (q < items) {
      int l, c0;
      place(q, l, c0);
      // position c0 + k + t - r lies in the line for t = r - c0 - k .. r + n - 1 - c0 - k
      const int t0 = !ADJ || c0 >= 0 ? 0 : max(0, r - c0 - (kOB - 1)) & ~3;
      const int t1 = !ADJ || c0 < n ? 2 * r + 1 : (r + n - c0 + 3) & ~3;
      conv_run(buf + l * pitch + c0 + front, w, t0, t1, acc[p]);
    }
  }
  __syncthreads();
#pragma unroll
  for (int p = 0; p < ROUNDS; ++p) {
    const int q = p * blockDim.x + threadIdx.x;
    if (q < items) {
      int l, c0;
      place(q, l, c0);
      f32x4* o = reinterpret_cast<f32x4*>(buf + l * pitch + lb.left * kOB + c0);
#pragma unroll
      for (int k = 0; k < kOB; k += 4) o[k / 4] = f32x4{acc[p][k], acc[p][k + 1], acc[p][k + 2], acc[p][k + 3]};
    }
  }
  __syncthreads();
  auto value = [&](int l, int j) {
    const float* C = buf + l * pitch + lb.left * kOB;
    float x = C[j];
    if (ADJ) {
      float m = 0.f;
      if (j > 0 && j <= r) m += C[-j];
      if (j < n - 1 && j >= n - 1 - r) m += C[2 * (n - 1) - j];
      x += m;
    }
    return x;
  };
  if (MU) {
    for (int q = threadIdx.x; q < n << sh; q += blockDim.x) {
      const int c = q & (lines - 1), j = q >> sh;
      if (c < held) out[base + (size_t)j * ns + c] = value(c, j);
    }
  } else {
    for (int l = 0; l < held; ++l)
      for (int q = threadIdx.x; q < n; q += blockDim.x) out[base + (size_t)l * ns + q] = value(l, q);
  }
}

size_t smooth_mu_lds_bytes(int n_theta, int r) {
  return (size_t)(r + 1 + (n_theta + 2 * r + 4) * kSmCols) * sizeof(float);
}

GaussTaps gauss_taps(double sigma, int r) {
  GaussTaps tp{};
  double sum = 0.0;
  for (int t = -r; t <= r; ++t) sum += std::exp(-0.5 * (t / sigma) * (t / sigma));
  for (int t = 0; t <= r; ++t) tp.w[t] = (float)(std::exp(-0.5 * (t / sigma) * (t / sigma)) / sum);
  return tp;
}

hipError_t launch_smooth(const Plan& p, const float* in, float* out, double sigma, int r, bool adjoint, int v0,
                         int nv, hipStream_t s) {
  const int K = p.kg.n_theta, S = p.kg.n_s;
  const GaussTaps tp = gauss_taps(sigma, r);
  auto pass = [&](auto adj, auto mu, const float* src) {
    constexpr bool ADJ = decltype(adj)::value, MU = decltype(mu)::value;
    const int n = MU ? K : S, per = LineBlocks(ADJ, n, r).all();
    auto lds = [&](int lines) { return (size_t)(tap_words(r) + lines * line_pitch(ADJ, n, r)) * sizeof(float); };
    int lines;
    if (MU) {
      // the most columns of which two workgroups share a CU's LDS and, in the transpose, whose
      // items one workgroup holds
      lines = 32;
      while (lines > 1 && (lds(lines) > kMaxLdsPerBlock / 2 || (ADJ && lines * per > 1024))) lines /= 2;
    } else {
      // as many rows as fill 512 threads
      lines = std::max(1, std::min(512 / per, 64));
      while (lines > 1 && lds(lines) > kMaxLdsPerBlock / 4) --lines;
    }
    const int strips = MU ? (S + lines - 1) / lines : 0;
    const unsigned grid = MU ? 8u * ((nv + 7) / 8) * strips : (unsigned)(((size_t)nv * K + lines - 1) / lines);
    const int threads = std::min(1024, (lines * per + 63) / 64 * 64);
    auto go = [&](auto rounds) {
      hipLaunchKernelGGL((k_smooth<ADJ, MU, decltype(rounds)::value>), dim3(grid), dim3(threads), lds(lines), s, src, out,
                         K, S, tp, r, v0, nv, lines, strips);
      return hipGetLastError();
    };
    // a row of up to 20351 bins (the Radon stage's limit) takes at most two rounds
    if (!MU && lines * per > 1024) return go(std::integral_constant<int, 2>{});
    return go(std::integral_constant<int, 1>{});
  };
  hipError_t e;
  if (!adjoint) {
    // G_mu G_s M: the s-pass into out, then the mu-pass in place
    if ((e = pass(std::false_type{}, std::false_type{}, in)) != hipSuccess) return e;
    return pass(std::false_type{}, std::true_type{}, out);
  }
  // (G_mu G_s)^T = G_s^T G_mu^T
  if ((e = pass(std::true_type{}, std::true_type{}, in)) != hipSuccess) return e;
  return pass(std::true_type{}, std::false_type{}, out);
}

}  // namespace dc
