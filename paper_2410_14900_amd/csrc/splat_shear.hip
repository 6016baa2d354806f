// The 2D Radon splat (A2d and the detector Radon, radon2d.hip's header) as a gather, for
// bins at least as wide as pixels and at most twice as wide.
//
// Take an angle's position t = l alpha + w beta + C with l the pixel index along the
// image axis on which t changes faster (|beta| <= |alpha|) and w the other one.  Row
// w is read shifted by a whole number of pixels sigma_w = rint(w beta / alpha), so
// the pixel that column l' holds, l = l' - sigma_w, stays near t = l' alpha + C.  A block of
// rows is taken in two sets (plan_host.h) over which a column's t covers at most one bin, so
// its hat function only ever meets three bins m-1, m, m+1.  With e = t - m in [-1, 1] their
// weights are (|e| - e)/2, 1 - |e| and (|e| + e)/2, so a column needs the sums
//   S0 = sum x,   S1 = sum e x,   H = sum |e| x.
// Neighbouring angles drift apart by a fraction of a pixel over a block, so G of them (the
// plan's choice, 4 at 360 angles) share sigma and the pixels read; e is linear in rho and w,
// so S0 and the two sums that make up S1 are common to them too, and each angle adds one FMA
// per pixel.  e depends on the geometry alone and is shared by four views, whose pixels lie
// side by side.  Per pixel-angle of a view that is 2 VALU operations (3/4 shared sums, 1/4
// position, 1 FMA) and 4 / G bytes from the vector caches, and about 0.7 operations for the
// end of each set, when the lanes add their sums to the sinogram rows in LDS as 32-bit
// fixed-point integers: results do not depend on the order and are bit-reproducible.  One
// LDS atomic per pixel-angle, which the scattering form (k_splat) needs, costs 9 clocks per
// wave and CU; a VALU operation 0.8.
//
// That is the float form, for the detector Radon into float32: its pixels are first rounded
// to the view's unit (the one k_splat uses), so that both forms sum the same numbers.
// dc_weight_radon, and results in 16 bits, take the exact form instead (k_splat_exact): the
// same walk, with k_splat's own two integers per pixel-angle, so its results are k_splat's bit
// for bit and do not depend on which of the two a plan takes.
//
// Half of the angles walk the image by columns and the shift makes lanes read any
// alignment of a row, so a first kernel rewrites the views once per call: weighted,
// converted to float32, four views interleaved, in row and in column order, with zero
// pixels around the rows.  The copy lives in the plan's workspace, a batch of views at a time.
//
// 496 views of 512^2 at 360 angles, with the maxima and the copy: k_splat 10.6 ms; float
// form 3.9 ms (3.4 vector operations per pixel-angle in all), exact form 6.1 ms (6.1).  Both
// issue 1.3 of them per clock and CU.
#include <algorithm>
#include <cmath>

#include "dc_internal.h"

namespace dc {

typedef float f32x4 __attribute__((ext_vector_type(4)));

static constexpr int kPad = kShearPad;
static constexpr int kVB = 4;                // views per record
static constexpr int kAhead = kShearAhead;
static constexpr int kGuard = kShearGuard;

// The copy of one view group: the row form (nv image rows, then zero rows up to rows[0]) and
// the column form, each kPad records, then its rows of n + kPad records
struct CopyShape {
  int nu, nv, rows[2];
  __host__ __device__ size_t form(int col) const {
    return (size_t)rows[col] * ((col ? nv : nu) + kPad) + kPad;
  }
  __host__ __device__ size_t group() const { return form(0) + form(1); }
};

// -------------------------------------------------------------------- copy
// One 32 x 32 tile of four views: both orders (the column order through LDS) of the weighted
// pixels w x; for the float form rounded to the view's unit, round(w x S) with
// S = qmax / (largest |w x| of the view); for the exact form, which scales while it sums,
// the views' largest |w x| are taken here (into vmax, zeroed before).  The tile grid
// covers kPad pixels past the image on both axes, which are written as zeros.  Bound by
// its writes (8 bytes for every 4 read).
template <typename Tin, bool WCOS, bool EXACT>
__global__ __launch_bounds__(256) void k_splat_copy(const Tin* __restrict__ img, f32x4* __restrict__ ws,
                                                    unsigned* __restrict__ vmax, KGrid g, CopyShape cs,
                                                    const float4* __restrict__ viewf, int v0, int nv, float qmax) {
  __shared__ f32x4 tile[32][33];
  __shared__ float tops[4][kVB];
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  const int gv = blockIdx.z * kVB;                   // first view of the group, from v0
  const size_t npix = (size_t)g.nu * g.nv;
  f32x4* rows = ws + (size_t)blockIdx.z * cs.group();
  f32x4* cols = rows + cs.form(0);
  float S[kVB], D[kVB];
#pragma unroll
  for (int b = 0; b < kVB; ++b) {
    const int vl = min(gv + b, nv - 1);
    const float vm = EXACT ? 0.f : __uint_as_float(vmax[vl]);
    S[b] = vm > 0.f ? qmax / vm : 0.f;
    D[b] = WCOS ? viewf[v0 + vl].x : 0.f;
  }
  const int i = blockIdx.x * 32 + tx;
  const float xu = (i - g.cu) * g.du;
  float top[kVB] = {};
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int jl = ty + 8 * q, j = blockIdx.y * 32 + jl;
    const bool in = i < g.nu && j < g.nv;
    const float yv = (j - g.cv) * g.dv;
    f32x4 x;
#pragma unroll
    for (int b = 0; b < kVB; ++b) {
      float p = in && gv + b < nv ? to_f32(img[(size_t)(v0 + gv + b) * npix + (size_t)j * g.nu + i]) : 0.f;
      // hardware rsqrt: the argument is at least D^2, far from the denormal range
      if (WCOS) p *= D[b] * __builtin_amdgcn_rsqf(fmaf(xu, xu, fmaf(yv, yv, D[b] * D[b])));
      x[b] = EXACT ? p : rintf(p * S[b]);
      if (EXACT) top[b] = fmaxf(top[b], fabsf(p));
    }
    tile[jl][tx] = x;
    if (i < g.nu + kPad && j < cs.rows[0]) rows[(size_t)j * (g.nu + kPad) + kPad + i] = x;
  }
  if (EXACT) {
#pragma unroll
    for (int m = 32; m > 0; m >>= 1)
#pragma unroll
      for (int b = 0; b < kVB; ++b) top[b] = fmaxf(top[b], __shfl_xor(top[b], m));
    if ((threadIdx.x & 63) == 0) {
#pragma unroll
      for (int b = 0; b < kVB; ++b) tops[threadIdx.x >> 6][b] = top[b];
    }
  }
  // the zero pixels before the first row of each form
  if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x < kPad) rows[threadIdx.x] = cols[threadIdx.x] = 0.f;
  __syncthreads();
  if (EXACT && threadIdx.x < kVB && gv + (int)threadIdx.x < nv) {
    const int b = threadIdx.x;   // magnitudes order like their bits
    const float t = fmaxf(fmaxf(tops[0][b], tops[1][b]), fmaxf(tops[2][b], tops[3][b]));
    if (t > 0.f) atomicMax(vmax + gv + b, __float_as_uint(t));
  }
  const int j = blockIdx.y * 32 + tx;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int il = ty + 8 * q, ic = blockIdx.x * 32 + il;
    if (j < g.nv + kPad && ic < cs.rows[1]) cols[(size_t)ic * (g.nv + kPad) + kPad + j] = tile[tx][il];
  }
}

// ------------------------------------------------------------------- gather
struct ShearArgs {
  CopyShape cs;
  int n_theta, ns, nsp;           // nsp: words between the sinogram rows in LDS
  int n_ang, n_views4, v0, views; // angle groups, view groups
  float scale, qmax;
};

// x rounded to the nearest integer (halves up), in one instruction
__device__ __forceinline__ int round_i32(float x) {
  int r;
  asm("v_cvt_rpi_i32_f32 %0, %1" : "=v"(r) : "v"(x));
  return r;
}

// One workgroup: four views, one group of up to G angles of one walk direction.  Its waves
// take the (block, column) pairs, 64 at a time, in turn and without barriers; a wave may hold
// the end of one block and the start of the next, since the blocks share the row table.
// Pixels are loaded kAhead rows ahead.
template <typename Tout, int G>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(6)))
void k_splat_float(const f32x4* ws, Tout* __restrict__ out, ShearArgs a, const ShearGroup* __restrict__ groups,
                   const ShearRow* __restrict__ steps, const unsigned* __restrict__ vmax_bits) {
  extern __shared__ int bins[];                // [G][kVB][nsp], kGuard words before bin 0
  __shared__ float sScale[kVB];
  // XCD x takes a contiguous eighth of the (view group, angle group) list, so the
  // workgroups that read one view group's copy share an L2
  const int total = a.n_views4 * a.n_ang, per = (total + 7) >> 3;
  const int job = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= per || job >= total) return;
  const int vg = job / a.n_ang, ag = job - vg * a.n_ang;
  const ShearGroup& gr = groups[ag];
  const int col = gr.col, kn = gr.kn, ns = a.ns;
  const int n = col ? a.cs.nv : a.cs.nu, walk = col ? a.cs.nu : a.cs.nv;
  const int pitch = n + kPad;
  const char* src = reinterpret_cast<const char*>(ws + (size_t)vg * a.cs.group() + (col ? a.cs.form(0) : 0));
  for (int q = threadIdx.x; q < kn * kVB * a.nsp; q += blockDim.x) bins[q] = 0;
  if ((int)threadIdx.x < kVB) {
    // |sum| per bin: the hat functions of one row's pixels add up to at most 3 - 2 |alpha|
    // (1 when |alpha| = 1), each at most qmax, over `walk` rows; 2^20 units to spare for rounding
    double al = 1.0;
    for (int g = 0; g < G; ++g) al = fmin(al, fabs(gr.a[g]));
    sScale[threadIdx.x] = (float)((2147483648.0 - 1048576.0) / ((3.0 - 2.0 * al) * walk * (double)a.qmax));
  }
  __syncthreads();
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int nw = blockDim.x >> 6;
  const ShearRow* rows = steps + ag * kShearPad;
  const int span = n + abs(gr.shift), left = min(gr.shift, 0);
  const int n_cols = gr.blocks * span;
  const int n_first = gr.n_first, n_rows = gr.rows;
  float half[kVB];   // half the scale of each view, in scalar registers
#pragma unroll
  for (int b = 0; b < kVB; ++b)
    half[b] = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(0.5f * sScale[b])));
  for (int c0 = wave * 64; c0 < n_cols; c0 += nw * 64) {
    // this lane's block and column l'; lanes past the last one repeat it and deposit nothing
    int blk = c0 / span, lp = c0 - blk * span + lane;
    if (span >= 64) {
      if (lp >= span) {
        lp -= span;
        ++blk;
      }
    } else {
      const int d = lp / span;
      blk += d;
      lp -= d * span;
    }
    const bool live = blk < gr.blocks;
    if (!live) {
      blk = gr.blocks - 1;
      lp = span - 1;
    }
    lp += left;
    unsigned off = (unsigned)((blk * n_rows * pitch + kPad + lp) * 16);
    // t of the column without the rest: its integer and its fraction
    float pf[G];
    int pi[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const double p = fma((double)lp, gr.a[g], fma((double)(blk * n_rows), gr.b[g], gr.base[g]));
      const double c = rint(p);
      pf[g] = (float)(p - c);
      pi[g] = (int)c;
    }
    auto load = [&](int row) { return *reinterpret_cast<const f32x4*>(src + row + off); };
    f32x4 x[kAhead];
#pragma unroll
    for (int w = 0; w < kAhead; ++w) {
      asm volatile("" ::: "memory");
      x[w] = load(gr.first[w]);
    }
    asm volatile("" ::: "memory");
    for (int set = 0; set < 2; ++set) {
      const int i1 = set ? n_rows : n_first;
      int i = set ? n_first : 0;
      if (i >= i1) continue;
      float e0[G];
      int mid[G];                          // the middle bin m
      f32x4 s0 = 0.f, m1 = 0.f, m2 = 0.f, h[G];
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const float fl = floorf(pf[g] + gr.lo[set][g]) + 1.0f;   // rest covers [lo, lo + 1): e in [-1, 1)
        e0[g] = pf[g] - fl;
        mid[g] = pi[g] + (int)fl;
        h[g] = 0.f;
      }
      ShearRow cur[kAhead], nxt[kAhead];   // scalar registers
#pragma unroll
      for (int w = 0; w < kAhead; ++w) {
        cur[w] = rows[i + w];
        asm volatile("" ::"s"(cur[w].rest[0]));   // wait for them here, not inside the loop
      }
      for (; i < i1; i += kAhead) {
        const int in = min(i + kAhead, n_rows - kAhead);   // the block's last step reads its own rows again
#pragma unroll
        for (int w = 0; w < kAhead; ++w) nxt[w] = rows[in + w];
#pragma unroll
        for (int w = 0; w < kAhead; ++w) {
          s0 += x[w];
#pragma unroll
          for (int b = 0; b < kVB; ++b) {
            m1[b] = fmaf(cur[w].wc, x[w][b], m1[b]);
            m2[b] = fmaf(cur[w].rho, x[w][b], m2[b]);
          }
#pragma unroll
          for (int g = 0; g < G; ++g) {
            const float e = e0[g] + cur[w].rest[g];
#pragma unroll
            for (int b = 0; b < kVB; ++b) h[g][b] = fmaf(x[w][b], fabsf(e), h[g][b]);
          }
          // the row is done with, and the loads stay here, kAhead rows before their use (the
          // compiler would put both off)
#pragma unroll
          for (int b = 0; b < kVB; ++b) {
            float t0 = s0[b], t1 = m1[b], t2 = m2[b], t3 = h[G - 1][b];
            asm volatile("" : "+v"(t0), "+v"(t1), "+v"(t2), "+v"(t3)::"memory");
            s0[b] = t0; m1[b] = t1; m2[b] = t2; h[G - 1][b] = t3;
          }
          x[w] = load(cur[w].ahead);
          asm volatile("" ::: "memory");
        }
#pragma unroll
        for (int w = 0; w < kAhead; ++w) cur[w] = nxt[w];
      }
      // the set's sums into the sinogram rows.  The scale is common to the group's angles,
      // so it is applied to the shared sums; bins outside the row go to its guard words
      float r0[kVB], r1[kVB], r2[kVB];
#pragma unroll
      for (int b = 0; b < kVB; ++b) {
        r0[b] = s0[b] * half[b];
        r1[b] = m1[b] * half[b];
        r2[b] = m2[b] * half[b];
      }
#pragma unroll
      for (int g = 0; g < G; ++g) {
        if (g >= kn) break;
        const int m = live ? min(max(mid[g], 1 - kGuard), ns + kGuard - 2) : 1 - kGuard;
        int* row = bins + (g * kVB * a.nsp + kGuard) + m;
#pragma unroll
        for (int b = 0; b < kVB; ++b) {
          const float s1 = fmaf(gr.alpha[g], r2[b], fmaf(gr.delta[g], r1[b], e0[g] * r0[b]));
          const float hh = h[g][b] * half[b];
          atomicAdd(row + b * a.nsp - 1, round_i32(hh - s1));
          atomicAdd(row + b * a.nsp, round_i32(2.0f * (r0[b] - hh)));
          atomicAdd(row + b * a.nsp + 1, round_i32(hh + s1));
        }
      }
    }
  }
  __syncthreads();
  // integers to values; consecutive threads write consecutive bins of one view's row
  const int k0 = gr.k0;
  for (int b = 0; b < kVB; ++b) {
    const int vl = vg * kVB + b;
    if (vl >= a.views) break;
    const float vm = __uint_as_float(vmax_bits[vl]), S = vm > 0.f ? a.qmax / vm : 0.f;
    const double inv = S > 0.f ? (double)a.scale / ((double)S * (double)sScale[b]) : 0.0;
    Tout* o = out + ((size_t)(a.v0 + vl) * a.n_theta + k0) * ns;
    for (int q = threadIdx.x; q < kn * ns; q += blockDim.x) {
      const int kk = q / ns, m = q - kk * ns;
      const int val = bins[(kk * kVB + b) * a.nsp + kGuard + m];
      o[q] = from_f32<Tout>((float)((double)val * inv));
    }
  }
}

// The exact form: the integer terms of k_splat, bit for bit.  A pixel x at fraction f (32.32
// fixed point, converted to float32) puts qa - qb on its bin and qb on the next: with
// xs = x S in float32, qa = round(x S), qb = round(xs f), rounded once each by adding 1.5 2^23.  Over a set of
// rows a column's pixels lie in bin m-1 or m; a pixel lies in bin m where its fraction is
// below phi, the fraction of the set's lower end.  So a column needs
//   A = sum qa,   N = sum over bin m-1 of (qa - qb),   P = sum over bin m of qb,
// as integers, and puts N, A - N - P and P on the bins m-1, m and m+1.  Per pixel-angle of a
// view: the rounding FMA and the two sums, each executed for its own lanes (3 operations:
// with -xs the FMA gives -qb, and qa - qb is one three-operand addition), 1 for the
// fraction and 3 / G for qa, A and xs.  The sums are of biased bit patterns; the lanes count P's terms.
static constexpr float kMagic = 12582912.0f;          // 1.5 * 2^23
static constexpr unsigned kMagicBits = 0x4B400000u;   // its bit pattern
static constexpr int kExactWaves = 4;                 // waves per SIMD

// p += y and ++count for the lanes with lo < phi, n += y + ya for the others (all lanes active
// on entry)
__device__ __forceinline__ void split_add(unsigned lo, unsigned phi, const unsigned (&y)[4], const unsigned (&ya)[4],
                                          unsigned (&p)[4], unsigned (&n)[4], unsigned& count) {
  unsigned c = count;
  unsigned p0 = p[0], p1 = p[1], p2 = p[2], p3 = p[3], n0 = n[0], n1 = n[1], n2 = n[2], n3 = n[3];
  asm volatile(
      "v_cmpx_lt_u32 vcc, %[lo], %[phi]\n\t"
      "v_add_u32 %[p0], %[y0], %[p0]\n\t"
      "v_add_u32 %[p1], %[y1], %[p1]\n\t"
      "v_add_u32 %[p2], %[y2], %[p2]\n\t"
      "v_add_u32 %[p3], %[y3], %[p3]\n\t"
      "v_add_u32 %[c], 1, %[c]\n\t"
      "s_not_b64 exec, exec\n\t"
      "v_add3_u32 %[n0], %[y0], %[a0], %[n0]\n\t"
      "v_add3_u32 %[n1], %[y1], %[a1], %[n1]\n\t"
      "v_add3_u32 %[n2], %[y2], %[a2], %[n2]\n\t"
      "v_add3_u32 %[n3], %[y3], %[a3], %[n3]\n\t"
      "s_mov_b64 exec, -1"
      : [p0] "+v"(p0), [p1] "+v"(p1), [p2] "+v"(p2), [p3] "+v"(p3), [n0] "+v"(n0), [n1] "+v"(n1), [n2] "+v"(n2),
        [n3] "+v"(n3), [c] "+v"(c)
      : [lo] "v"(lo), [phi] "v"(phi), [y0] "v"(y[0]), [y1] "v"(y[1]), [y2] "v"(y[2]), [y3] "v"(y[3]), [a0] "v"(ya[0]),
        [a1] "v"(ya[1]), [a2] "v"(ya[2]), [a3] "v"(ya[3])
      : "scc", "vcc");
  count = c;
  p[0] = p0; p[1] = p1; p[2] = p2; p[3] = p3;
  n[0] = n0; n[1] = n1; n[2] = n2; n[3] = n3;
}

template <typename Tout, int G>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(kExactWaves)))
void k_splat_exact(const f32x4* ws, Tout* __restrict__ out, ShearArgs a, const double* __restrict__ angd,
                   const ShearGroup* __restrict__ groups, const ShearRow* __restrict__ steps,
                   const unsigned* __restrict__ vmax_bits) {
  typedef unsigned frac_t __attribute__((ext_vector_type(G)));
  extern __shared__ int bins[];   // [G][kVB][nsp], kGuard words before bin 0; then the fractions [n + 2 kPad][G]
  const int total = a.n_views4 * a.n_ang, per = (total + 7) >> 3;
  const int job = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= per || job >= total) return;
  const int vg = job / a.n_ang, ag = job - vg * a.n_ang;
  const ShearGroup& gr = groups[ag];
  const int col = gr.col, kn = gr.kn, ns = a.ns;
  const int n = col ? a.cs.nv : a.cs.nu;
  const int pitch = n + kPad;
  const char* src = reinterpret_cast<const char*>(ws + (size_t)vg * a.cs.group() + (col ? a.cs.form(0) : 0));
  float S[kVB], T[kVB];   // scalar registers
#pragma unroll
  for (int b = 0; b < kVB; ++b) {
    const float vm = __uint_as_float(vmax_bits[min(vg * kVB + b, a.views - 1)]);
    S[b] = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(vm > 0.f ? a.qmax / vm : 0.f)));
    T[b] = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(S[b] * -2.3283064365386963e-10f)));   // 2^-32
  }
  for (int q = threadIdx.x; q < kn * kVB * a.nsp; q += blockDim.x) bins[q] = 0;
  // low words of t(l, row 0) in 32.32 fixed point, rounded as k_splat rounds them
  unsigned* frac = reinterpret_cast<unsigned*>(bins + G * kVB * a.nsp);
  for (int q = threadIdx.x; q < G * (n + 2 * kPad); q += blockDim.x) {
    const int l = q / G, k = gr.k0 + min(q - l * G, kn - 1);
    const double t0 = fma((double)(l - kPad), angd[3 * k + col], angd[3 * k + 2]);
    frac[q] = (unsigned)((t0 - floor(t0)) * 4294967296.0);
  }
  __syncthreads();
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int nw = blockDim.x >> 6;
  const ShearRow* rows = steps + ag * kShearPad;
  const int span = n + abs(gr.shift), left = min(gr.shift, 0);
  const int n_cols = gr.blocks * span;
  const int n_first = gr.n_first, n_rows = gr.rows;
  for (int c0 = wave * 64; c0 < n_cols; c0 += nw * 64) {
    // this lane's block and column l'; lanes past the last one repeat it and deposit nothing
    int blk = c0 / span, lp = c0 - blk * span + lane;
    if (span >= 64) {
      if (lp >= span) {
        lp -= span;
        ++blk;
      }
    } else {
      const int d = lp / span;
      blk += d;
      lp -= d * span;
    }
    const bool live = blk < gr.blocks;
    if (!live) {
      blk = gr.blocks - 1;
      lp = span - 1;
    }
    lp += left;
    const unsigned off = (unsigned)((blk * n_rows * pitch + kPad + lp) * 16);
    const frac_t* fcol = reinterpret_cast<const frac_t*>(frac) + kPad + lp;
    float pf[G];
    int pi[G];
    unsigned fblk[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const double p = fma((double)lp, gr.a[g], fma((double)(blk * n_rows), gr.b[g], gr.base[g]));
      const double c = rint(p);
      pf[g] = (float)(p - c);
      pi[g] = (int)c;
      fblk[g] = (unsigned)blk * gr.block_step[g];
    }
    auto load = [&](int row) { return *reinterpret_cast<const f32x4*>(src + row + off); };
    f32x4 x[kAhead];
#pragma unroll
    for (int w = 0; w < kAhead; ++w) {
      asm volatile("" ::: "memory");
      x[w] = load(gr.first[w]);
    }
    asm volatile("" ::: "memory");
    for (int set = 0; set < 2; ++set) {
      const int i0 = set ? n_first : 0, i1 = set ? n_rows : n_first;
      if (i0 >= i1) continue;
      int mid[G];
      unsigned phi[G], cnt[G], A[kVB], P[G][kVB], N[G][kVB];
#pragma unroll
      for (int g = 0; g < G; ++g) {
        // the set covers less than 1 - 1e-5 bins from its lower end: 5e-6 of margin on both sides
        const float lo = pf[g] + gr.lo[set][g] - 5e-6f, fl = floorf(lo);
        mid[g] = pi[g] + (int)fl + 1;
        phi[g] = (unsigned)((lo - fl) * 4294967296.0f);
        cnt[g] = 0u;
#pragma unroll
        for (int b = 0; b < kVB; ++b) P[g][b] = N[g][b] = 0u;
      }
#pragma unroll
      for (int b = 0; b < kVB; ++b) A[b] = 0u;
      ShearRow cur[kAhead], nxt[kAhead];   // scalar registers
#pragma unroll
      for (int w = 0; w < kAhead; ++w) {
        cur[w] = rows[i0 + w];
        asm volatile("" ::"s"(cur[w].step[0]));   // wait for them here, not inside the loop
      }
      for (int i = i0; i < i1; i += kAhead) {
        const int in = min(i + kAhead, n_rows - kAhead);   // the block's last step reads its own rows again
#pragma unroll
        for (int w = 0; w < kAhead; ++w) nxt[w] = rows[in + w];
#pragma unroll
        for (int w = 0; w < kAhead; ++w) {
          const frac_t f = *(fcol - cur[w].sigma);
          unsigned ya[kVB];
          f32x4 xs;
#pragma unroll
          for (int b = 0; b < kVB; ++b) {
            ya[b] = __float_as_uint(fmaf(x[w][b], S[b], kMagic));
            A[b] += ya[b];
            xs[b] = x[w][b] * T[b];   // -xs 2^-32
          }
#pragma unroll
          for (int g = 0; g < G; ++g) {
            const unsigned lo = f[g] + fblk[g] + cur[w].step[g];
            const float fl = (float)lo;
            unsigned y[kVB];   // bits of magic - qb
#pragma unroll
            for (int b = 0; b < kVB; ++b) y[b] = __float_as_uint(fmaf(xs[b], fl, kMagic));
            split_add(lo, phi[g], y, ya, P[g], N[g], cnt[g]);
          }
#pragma unroll
          for (int b = 0; b < kVB; ++b) asm volatile("" : "+v"(A[b])::"memory");
          // the loads stay here, kAhead rows before their use (the compiler would put them off)
          x[w] = load(cur[w].ahead);
          asm volatile("" ::: "memory");
        }
#pragma unroll
        for (int w = 0; w < kAhead; ++w) cur[w] = nxt[w];
      }
      // the set's sums into the sinogram rows; bins outside the row go to its guard words
      const unsigned abias = (unsigned)(i1 - i0) * kMagicBits;
#pragma unroll
      for (int g = 0; g < G; ++g) {
        if (g >= kn) break;
        const int m = live ? min(max(mid[g], 1 - kGuard), ns + kGuard - 2) : 1 - kGuard;
        unsigned* row = reinterpret_cast<unsigned*>(bins) + (g * kVB * a.nsp + kGuard) + m;
        const unsigned pbias = cnt[g] * kMagicBits;
        const unsigned nbias = ((unsigned)(i1 - i0) - cnt[g]) * (2u * kMagicBits);
#pragma unroll
        for (int b = 0; b < kVB; ++b) {
          const unsigned p = pbias - P[g][b], q = N[g][b] - nbias;
          atomicAdd(row + b * a.nsp - 1, q);
          atomicAdd(row + b * a.nsp, A[b] - abias - q - p);
          atomicAdd(row + b * a.nsp + 1, p);
        }
      }
    }
  }
  __syncthreads();
  // integers to values; consecutive threads write consecutive bins of one view's row
  const int k0 = gr.k0;
  for (int b = 0; b < kVB; ++b) {
    const int vl = vg * kVB + b;
    if (vl >= a.views) break;
    const float vm = __uint_as_float(vmax_bits[vl]), S = vm > 0.f ? a.qmax / vm : 0.f;
    const double inv = S > 0.f ? (double)a.scale / (double)S : 0.0;
    Tout* o = out + ((size_t)(a.v0 + vl) * a.n_theta + k0) * ns;
    for (int q = threadIdx.x; q < kn * ns; q += blockDim.x) {
      const int kk = q / ns, m = q - kk * ns;
      o[q] = from_f32<Tout>((float)((double)bins[(kk * kVB + b) * a.nsp + kGuard + m] * inv));
    }
  }
}

// ---------------------------------------------------------------- dispatch
// The workspace holds at most about this many bytes; larger calls take several batches
static constexpr size_t kShearWorkBytes = (size_t)512 << 20;

static CopyShape copy_shape(const Plan& p) { return {p.kg.nu, p.kg.nv, {p.shear_pad_rows[0], p.shear_pad_rows[1]}}; }

size_t splat_shear_workspace(const Plan& p) {
  const size_t per4 = copy_shape(p).group() * 16;    // four views
  return std::max<size_t>(1, std::min<size_t>((p.n_views + 3) / 4, kShearWorkBytes / per4)) * per4;
}

// `exact`: the integer terms of k_splat (bit-identical); otherwise float32 sums of the
// pixels rounded to its unit.  vmax: words of the views' largest magnitudes, zero for the exact form and formed
// for the other.
hipError_t launch_splat_shear(const Plan& p, const void* img, dc_dtype t_in, bool wcos, float scale, void* out,
                              dc_dtype t_out, int v0, int nv, bool exact, hipStream_t s, unsigned* vmax) {
  const CopyShape cs = copy_shape(p);
  // equal batches of view groups
  const int all = (nv + 3) / 4;
  const int cap = std::max(1, (int)(p.splat_ws_bytes / (cs.group() * 16)));
  const int n_batches = (all + cap - 1) / cap;
  const int batch = (all + n_batches - 1) / n_batches;
  const int nsp = shear_row_words(p.kg.n_s), nmax = std::max(p.kg.nu, p.kg.nv);
  const size_t rows_lds = (size_t)p.shear_g * kVB * nsp * sizeof(int);
  const size_t frac_lds = (size_t)p.shear_g * (nmax + 2 * kPad) * sizeof(unsigned);
  const int items = (int)((size_t)p.kg.nu * p.kg.nv / 64 / 32) + 1;
  for (int b0 = 0; b0 < all; b0 += batch) {
    const int groups = std::min(batch, all - b0), vb = 4 * b0, bn = std::min(4 * groups, nv - vb);
    const dim3 cgrid((std::max(p.kg.nu + kPad, cs.rows[1]) + 31) / 32, (std::max(p.kg.nv + kPad, cs.rows[0]) + 31) / 32,
                     groups);
    hipError_t e = by_dtype(t_in, [&](auto tin) {
      using Tin = decltype(tin);
      auto go = [&](auto w, auto x) {
        hipLaunchKernelGGL((k_splat_copy<Tin, decltype(w)::value, decltype(x)::value>), cgrid, dim3(256), 0, s,
                           (const Tin*)img, (f32x4*)p.d_splat_ws, vmax + vb, p.kg, cs, (const float4*)p.d_view, v0 + vb,
                           bn, p.splat_qmax);
      };
      if (wcos) go(std::true_type{}, std::true_type{});
      else if (exact) go(std::false_type{}, std::true_type{});
      else go(std::false_type{}, std::false_type{});
      return hipGetLastError();
    });
    if (e != hipSuccess) return e;
    const ShearArgs a{cs, p.kg.n_theta, p.kg.n_s, nsp, p.shear_groups, groups, v0 + vb, bn, scale, p.splat_qmax};
    e = by_dtype(t_out, [&](auto tout) {
      using Tout = decltype(tout);
      auto by_g = [&](auto&& f) {
        if (p.shear_g == 4) f(std::integral_constant<int, 4>{});
        else if (p.shear_g == 2) f(std::integral_constant<int, 2>{});
        else f(std::integral_constant<int, 1>{});
      };
      if (exact) {
        // two workgroups of kExactWaves waves per SIMD between them share a CU where its LDS
        // allows and there are enough of them
        const size_t lds = rows_lds + frac_lds;
        const int total = groups * p.shear_groups;
        const int waves = std::min(items, 2 * (lds + 1024) <= (size_t)kLdsPerWorkgroup && total >= 512 ? 2 * kExactWaves : 16);
        const dim3 grid(8 * ((total + 7) / 8));
        by_g([&](auto g) {
          hipLaunchKernelGGL((k_splat_exact<Tout, decltype(g)::value>), grid, dim3(64 * waves), lds, s,
                             (const f32x4*)p.d_splat_ws, (Tout*)out, a, p.d_ang, p.d_shear_groups, p.d_shear_rows,
                             vmax + vb);
        });
        return hipGetLastError();
      }
      // 8 waves per workgroup while three of them (24 waves of 80 registers) fit a CU's LDS
      // and there are enough of them; otherwise 16
      const int total = groups * p.shear_groups;
      const int waves = std::min(items, 3 * (rows_lds + 1024) <= (size_t)kLdsPerWorkgroup && total >= 512 ? 8 : 16);
      const dim3 grid(8 * ((total + 7) / 8));
      by_g([&](auto g) {
        hipLaunchKernelGGL((k_splat_float<Tout, decltype(g)::value>), grid, dim3(64 * waves), rows_lds, s,
                           (const f32x4*)p.d_splat_ws, (Tout*)out, a, p.d_shear_groups, p.d_shear_rows, vmax + vb);
      });
      return hipGetLastError();
    });
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace dc
