// Structural similarity of two volumes (the SSIM term of the training loss, eq. 13)
// and its gradient w.r.t. the first volume.
//
// Standard definition in 3D: window moments mu_x = G*x, mu_y = G*y, E[x^2], E[y^2],
// E[xy] with the normalised Gaussian window G (sigma 1.5, 11 taps per axis) at the
// positions where the whole window lies inside the volume ("valid" grid),
//   S = (2 mu_x mu_y + C1)(2 s_xy + C2) / ((mu_x^2 + mu_y^2 + C1)(s_xx + s_yy + C2)),
// SSIM = mean S.  The gradient spreads the per-position derivatives of S w.r.t.
// (mu_x, E[x^2], E[xy]) back over the windows (the transposed valid convolution,
// zero outside) and combines them as (T0 + 2 x T1 + y T2) / N.
//
// The separable passes run z, y, x and back x, y, z, each rounded to float32, in three
// kernels over a caller-provided workspace: z and y (five moments), a row's x pass, map and
// transposed x pass, and the transposed y and z passes.  That is 18 volumes of memory traffic
// (read x, y; 5 fields out and in; 3 out and in; read x, y; write the gradient) where one
// kernel per pass took 49: 256^3 with gradient 2.01 -> 0.74 ms.  The mean is reduced in a fixed order
// (per-block partial sums, then one block), so results are bit-reproducible.
#include <algorithm>
#include <cmath>

#include "dc_internal.h"

namespace dc {

static constexpr int kSsR = 5, kSsT = 2 * kSsR + 1;
struct SsimWindow {
  float w[kSsT];
};

static SsimWindow ssim_window() {
  SsimWindow s{};
  double sum = 0.0, v[kSsT];
  for (int t = 0; t < kSsT; ++t) sum += (v[t] = std::exp(-0.5 * ((t - kSsR) / 1.5) * ((t - kSsR) / 1.5)));
  for (int t = 0; t < kSsT; ++t) s.w[t] = (float)(v[t] / sum);
  return s;
}

// z and y passes of the five moments of x and y (mu_x, mu_y, E[x^2], E[y^2], E[xy]):
// out [5][nz-10][ny-10][nx].  A workgroup owns 64 x, kMomY outputs in y and zc <= kMomZ in z: its 16
// waves hold kMomY + 10 rows' runs along z in registers, two rows each, and per output plane
// leave the z pass of all rows in LDS, from which 15 of them form the y pass, a field and
// eight consecutive y each.  Bound by vector operations (a third of them for the products
// and the halo rows).
static constexpr int kMomZ = 6, kMomY = 22, kMomRows = kMomY + 2 * kSsR;
__global__ __launch_bounds__(1024) void k_ss_moments(const float* __restrict__ x, const float* __restrict__ y,
                                                     float* __restrict__ out, int nz, int ny, int nx, int zc,
                                                     SsimWindow W) {
  __shared__ float m[2][5][kMomRows][64];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i = blockIdx.x * 64 + lane, y0 = blockIdx.y * kMomY, z0 = blockIdx.z * zc;
  const int vz = nz - 2 * kSsR, vy = ny - 2 * kSsR;
  const size_t plane = (size_t)ny * nx, n_out = (size_t)vz * vy * nx;
  const int ic = min(i, nx - 1);
  constexpr int kRun = kMomZ + 2 * kSsR;
  float xv[2][kRun], yv[2][kRun];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const size_t at = (size_t)min(y0 + wave + 16 * h, ny - 1) * nx + ic;
#pragma unroll
    for (int t = 0; t < kRun; ++t) {
      const size_t q = (size_t)min(z0 + t, nz - 1) * plane + at;
      xv[h][t] = x[q];
      yv[h][t] = y[q];
    }
  }
#pragma unroll
  for (int u = 0; u < kMomZ; ++u) {
    if (u >= zc || z0 + u >= vz) break;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      float a[5] = {0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int t = 0; t < kSsT; ++t) {
        const float xt = xv[h][u + t], yt = yv[h][u + t], wt = W.w[t];
        a[0] = fmaf(wt, xt, a[0]);
        a[1] = fmaf(wt, yt, a[1]);
        a[2] = fmaf(wt, xt * xt, a[2]);
        a[3] = fmaf(wt, yt * yt, a[3]);
        a[4] = fmaf(wt, xt * yt, a[4]);
      }
#pragma unroll
      for (int f = 0; f < 5; ++f) m[u & 1][f][wave + 16 * h][lane] = a[f];
    }
    __syncthreads();
    if (wave < 15) {
      const int f = wave / 3, r0 = wave % 3 * 8;
      float v[8 + 2 * kSsR];
#pragma unroll
      for (int t = 0; t < 8 + 2 * kSsR; ++t) v[t] = m[u & 1][f][min(r0 + t, kMomRows - 1)][lane];
      float* o = out + f * n_out + (size_t)(z0 + u) * vy * nx + i;
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        float a = 0.f;
#pragma unroll
        for (int t = 0; t < kSsT; ++t) a = fmaf(W.w[t], v[k + t], a);
        const int r = r0 + k;
        if (r < kMomY && y0 + r < vy && i < nx) o[(size_t)(y0 + r) * nx] = a;
      }
    }
  }
}

// x pass, SSIM map and, WANT_GRAD, transposed x pass of `rows` rows: mom [5][n_rows][nx] in,
// per-workgroup sums of S (fixed-order tree) into part[], the derivative fields
// (dS/dmu_x, dS/dE[x^2], dS/dE[xy]) convolved along x into d [3][n_rows][nx].  Four
// consecutive positions per thread from windows of 14, all in LDS; rows longer than kRowChunk
// in chunks (blockIdx.y), which form the 10 derivatives before their own again.
// lds = moments [rows][5][pitch], derivatives [rows][3][dpitch] with zeros around them
static constexpr int kRowChunk = 1024;
static __host__ __device__ int ss_pitch(int chunk) { return (chunk + 3) / 4 * 4 + 28; }
static __host__ __device__ int ss_dpitch(int chunk) { return (chunk + 3) / 4 * 4 + 32; }

// kSsT taps, in order, of four positions from the window at v (16-byte aligned); BACK: position
// k takes v[k + 12 - t], otherwise v[k + t]
template <bool BACK>
__device__ __forceinline__ void ss_conv4(const float* __restrict__ v, const SsimWindow& W, float (&a)[4]) {
  float win[16];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const float4 p = reinterpret_cast<const float4*>(v)[q];
    win[4 * q] = p.x; win[4 * q + 1] = p.y; win[4 * q + 2] = p.z; win[4 * q + 3] = p.w;
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) a[k] = 0.f;
#pragma unroll
  for (int t = 0; t < kSsT; ++t)
#pragma unroll
    for (int k = 0; k < 4; ++k) a[k] = fmaf(W.w[t], win[BACK ? k + 12 - t : k + t], a[k]);
}

template <bool WANT_GRAD>
__global__ __launch_bounds__(256) void k_ss_rows(const float* __restrict__ mom, int n_rows, int nx, int rows, float C1,
                                                 float C2, double* __restrict__ part, float* __restrict__ d,
                                                 SsimWindow W) {
  extern __shared__ float sm[];
  __shared__ double red[256];
  const int chunk = min(nx, kRowChunk), x0 = blockIdx.y * chunk, x1 = min(nx, x0 + chunk);
  const int vx = nx - 2 * kSsR, pitch = ss_pitch(chunk), dpitch = ss_dpitch(chunk);
  const int o = max(0, x0 - 12), jend = min(vx, x1);   // valid positions formed here: o .. jend - 1
  const int r0 = blockIdx.x * rows, held = min(rows, n_rows - r0);
  float* der = sm + rows * 5 * pitch;   // position j of the valid row at der[.. + 12 + j - o]
  const size_t n_in = (size_t)n_rows * nx;
  // word q = l pitch + m of the moments, l = f held + r; a thread's words lie blockDim.x apart, so
  // (l, m) advances with one carry, and eight are on their way at a time
  {
    const int dl = blockDim.x / pitch, dm = blockDim.x - dl * pitch, total = held * 5 * pitch;
    int l = threadIdx.x / pitch, m = threadIdx.x - l * pitch;
    constexpr int kLoad = 8;
    for (int q0 = threadIdx.x; q0 < total; q0 += kLoad * blockDim.x) {
      float v[kLoad];
      int at[kLoad];
#pragma unroll
      for (int u = 0; u < kLoad; ++u) {
        int f = 0;   // l / held
#pragma unroll
        for (int g = 1; g < 5; ++g) f += l >= g * held;
        const int r = l - f * held;
        at[u] = (r * 5 + f) * pitch + m;
        v[u] = l < 5 * held && o + m < nx ? mom[f * n_in + (size_t)(r0 + r) * nx + o + m] : 0.f;
        l += dl;
        m += dm;
        if (m >= pitch) {
          m -= pitch;
          ++l;
        }
      }
#pragma unroll
      for (int u = 0; u < kLoad; ++u)
        if (q0 + u * (int)blockDim.x < total) sm[at[u]] = v[u];
    }
  }
  if (WANT_GRAD)
    for (int q = threadIdx.x; q < rows * 3 * dpitch; q += blockDim.x) der[q] = 0.f;
  __syncthreads();
  double s = 0.0;
  const int blocks = max(0, (jend - o + 3) / 4);
  for (int q = threadIdx.x; q < held * blocks; q += blockDim.x) {
    const int r = q / blocks, l0 = (q - r * blocks) * 4;
    float m[5][4];
#pragma unroll
    for (int f = 0; f < 5; ++f) ss_conv4<false>(sm + (r * 5 + f) * pitch + l0, W, m[f]);
    float* dr = der + r * 3 * dpitch + 12 + l0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (o + l0 + k >= jend) break;
      const float mx = m[0][k], my = m[1][k], exx = m[2][k], eyy = m[3][k], exy = m[4][k];
      const float A1 = 2.f * mx * my + C1, A2 = 2.f * (exy - mx * my) + C2;
      const float B1 = mx * mx + my * my + C1, B2 = (exx - mx * mx) + (eyy - my * my) + C2;
      const float inv = 1.f / (B1 * B2);
      const float S = A1 * A2 * inv;
      if (o + l0 + k >= x0) s += (double)S;
      if (WANT_GRAD) {
        dr[k] = 2.f * my * (A2 - A1) * inv - 2.f * mx * S * (1.f / B1 - 1.f / B2);
        dr[dpitch + k] = -S / B2;
        dr[2 * dpitch + k] = 2.f * A1 * inv;
      }
    }
  }
  red[threadIdx.x] = s;
  __syncthreads();
  if (WANT_GRAD) {
    const int oblocks = (x1 - x0 + 3) / 4;
    for (int q = threadIdx.x; q < held * 3 * oblocks; q += blockDim.x) {
      const int l = q / oblocks, i0 = x0 + (q - l * oblocks) * 4, r = l / 3, f = l - 3 * r;
      float a[4];
      // position i takes der[i - t], at row[12 + i - o - t]
      ss_conv4<true>(der + l * dpitch + i0 - o, W, a);
      float* out = d + f * n_in + (size_t)(r0 + r) * nx + i0;
      if (nx % 4 == 0) {
        *reinterpret_cast<float4*>(out) = make_float4(a[0], a[1], a[2], a[3]);
      } else {
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (i0 + k < x1) out[k] = a[k];
      }
    }
  }
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.y * gridDim.x + blockIdx.x] = red[0];
}

// transposed y and z passes of the derivative fields d [3][nz-10][ny-10][nx], combined into
// the gradient: grad = (T0 + 2 x T1 + y T2) / N.  A workgroup owns 64 x, 16 y (a wave each) and
// zc z: plane by plane the rows that its y pass needs are staged in LDS (two planes ahead in
// registers), and each thread keeps its column's last 11 planes of the y pass in a ring of
// registers for the z pass.
static constexpr int kGradY = 16, kGradRows = kGradY + 2 * kSsR;
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(4)))
void k_ss_grad(const float* __restrict__ d, const float* __restrict__ x, const float* __restrict__ y,
               float* __restrict__ grad, int nz, int ny, int nx, int zc, float invN, SsimWindow W) {
  __shared__ float rows[2][3][kGradRows][64];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i = blockIdx.x * 64 + lane, y0 = blockIdx.y * kGradY, z0 = blockIdx.z * zc;
  const int vz = nz - 2 * kSsR, vy = ny - 2 * kSsR;
  const size_t vplane = (size_t)vy * nx, n_in = vz * vplane;
  const int ic = min(i, nx - 1), iy = y0 + wave, iyc = min(iy, ny - 1);
  const int planes = min(zc, nz - z0) + 2 * kSsR;   // jz = z0 - 10 .. z0 + zc - 1
  constexpr int kLoads = (3 * kGradRows + 15) / 16;
  float stg[2][kLoads];
  auto fetch = [&](int p, float (&to)[kLoads]) {   // rows y0 - 10 .. y0 + 15 of plane z0 - 10 + p; zero outside
    const int jz = z0 - 2 * kSsR + p;
    const float* plane = d + min(max(jz, 0), vz - 1) * vplane;
#pragma unroll
    for (int l = 0; l < kLoads; ++l) {
      const int q = min(wave + 16 * l, 3 * kGradRows - 1), f = q / kGradRows, jy = y0 - 2 * kSsR + q - f * kGradRows;
      const float v = plane[f * n_in + (size_t)min(max(jy, 0), vy - 1) * nx + ic];
      to[l] = (unsigned)jy < (unsigned)vy && (unsigned)jz < (unsigned)vz ? v : 0.f;
    }
  };
  float c[kSsT][3];
  fetch(0, stg[0]);
  fetch(1, stg[1]);
  // plane p = p0 + r: ring slot r of 11, staging buffers by the parity of p (22 planes a turn)
  for (int p0 = 0; p0 < planes; p0 += 2 * kSsT) {
#pragma unroll
    for (int r = 0; r < 2 * kSsT; ++r) {
      const int p = p0 + r;
      if (p >= planes) break;
#pragma unroll
      for (int l = 0; l < kLoads; ++l) {
        const int q = wave + 16 * l;
        if (q < 3 * kGradRows) (&rows[r & 1][0][0][0])[q * 64 + lane] = stg[r & 1][l];
      }
      __syncthreads();
      // the output plane's own volumes, on their way during the y pass (loads return in order:
      // ahead of the next rows)
      const int iz = z0 + p - 2 * kSsR;
      const size_t q = ((size_t)max(iz, 0) * ny + iyc) * nx + ic;
      const float xq = x[q], yq = y[q];
      asm volatile("" ::: "memory");
      fetch(p + 2, stg[r & 1]);
      asm volatile("" ::: "memory");
#pragma unroll
      for (int f = 0; f < 3; ++f) {
        float a = 0.f;
#pragma unroll
        for (int t = 0; t < kSsT; ++t) a = fmaf(W.w[t], rows[r & 1][f][wave + 2 * kSsR - t][lane], a);
        c[r % kSsT][f] = a;
      }
      if (p >= 2 * kSsR) {
        float a[3] = {0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < kSsT; ++t)
#pragma unroll
          for (int f = 0; f < 3; ++f) a[f] = fmaf(W.w[t], c[(r + kSsT - t) % kSsT][f], a[f]);
        if (iy < ny && i < nx) grad[q] = (a[0] + 2.f * xq * a[1] + yq * a[2]) * invN;
      }
    }
  }
}

__global__ __launch_bounds__(1024) void k_ss_mean(const double* __restrict__ part, int nb, double invN,
                                                 float* __restrict__ out) {
  __shared__ double red[1024];
  double s = 0.0;
  for (int i = threadIdx.x; i < nb; i += blockDim.x) s += part[i];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 512; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = (float)(red[0] * invN);
}

size_t ssim_workspace_bytes(int nz, int ny, int nx) {
  const size_t a = (size_t)(nz - 2 * kSsR) * ny * nx;   // after the z pass
  // room for 10 fields of that size and 1024 sums: callers may keep a workspace they sized
  // once; 8 fields and a sum per few rows of it are used
  return 2 * 5 * a * sizeof(float) + 1024 * sizeof(double) + 256;
}

hipError_t launch_ssim(const float* x, const float* y, int nz, int ny, int nx, float L, float* ssim, float* grad,
                       void* work, hipStream_t s) {
  const SsimWindow W = ssim_window();
  const int vz = nz - 2 * kSsR, vy = ny - 2 * kSsR, vx = nx - 2 * kSsR;
  const size_t a = (size_t)vz * ny * nx, c = (size_t)vz * vy * vx;
  const int n_rows = vz * vy;
  // rows of up to 256 threads' worth, in a quarter of a CU's LDS (with the derivatives, so that
  // the sums are grouped alike without them)
  const int chunk = std::min(nx, kRowChunk), chunks = (nx + chunk - 1) / chunk;
  auto lds = [&](int rows) { return (size_t)rows * (5 * ss_pitch(chunk) + 3 * ss_dpitch(chunk)) * sizeof(float); };
  int rows = std::max(1, 256 / ((chunk + 3) / 4));
  while (rows > 1 && lds(rows) > kMaxLdsPerBlock / 4) --rows;
  const int blocks = (n_rows + rows - 1) / rows;
  float* mom = (float*)work;          // [5][vz][vy][nx]
  float* d = mom + 5 * a;             // [3][vz][vy][nx]
  double* part = (double*)(d + 3 * a);   // [blocks]: at most 2 a floats
  const float C1 = (0.01f * L) * (0.01f * L), C2 = (0.03f * L) * (0.03f * L);
  const int gx = (nx + 63) / 64, my = (vy + kMomY - 1) / kMomY;
  // fewer planes per workgroup while that leaves CUs idle (one workgroup per CU)
  const int mz = std::max(1, std::min(kMomZ, (int)(((size_t)vz * gx * my + 255) / 256)));
  hipLaunchKernelGGL(k_ss_moments, dim3(gx, my, (vz + mz - 1) / mz), dim3(1024), 0, s, x, y, mom, nz, ny, nx, mz, W);
  if (grad)
    hipLaunchKernelGGL(k_ss_rows<true>, dim3(blocks, chunks), dim3(256), lds(rows), s, mom, n_rows, nx, rows, C1, C2, part, d, W);
  else
    hipLaunchKernelGGL(k_ss_rows<false>, dim3(blocks, chunks), dim3(256), lds(rows), s, mom, n_rows, nx, rows, C1, C2, part, d, W);
  hipLaunchKernelGGL(k_ss_mean, dim3(1), dim3(1024), 0, s, part, blocks * chunks, 1.0 / (double)c, ssim);
  if (grad) {
    // zc outputs cost zc + 10 planes: as few as keep the workgroups at two per CU, and 34
    // (two turns of the ring) at most
    const int gy = (ny + kGradY - 1) / kGradY;
    const int zc = std::max(2, std::min(34, (int)(((size_t)nz * gx * gy + 511) / 512)));
    hipLaunchKernelGGL(k_ss_grad, dim3(gx, gy, (nz + zc - 1) / zc), dim3(1024), 0, s, d, x, y, grad, nz, ny, nx, zc,
                       (float)(1.0 / (double)c), W);
  }
  return hipGetLastError();
}

}  // namespace dc
