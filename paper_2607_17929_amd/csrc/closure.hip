// Learned force closure: a 3-layer 3x3x3 convolutional network on the mesh.
//
// Not part of the paper's method.  The network maps fields of the particle-mesh
// solution (density contrast, gradient of phi) to a correction of the gathered
// force; it is trained on pairs of the same particles' forces from a mesh and a
// mesh of twice the resolution.  conv(4->16)-ReLU-conv(16->16)-ReLU-conv(16->3),
// periodic padding, taps d in {-1,0,1}^3 (cross-correlation).
//
// Every layer runs as a 16 -> 16 channel convolution (the 4 input and 3 output
// channels are zero-padded) on channels-last bfloat16 activations
// [z][y][x][16] with FP32 accumulation on the matrix cores: an implicit GEMM
// whose M dimension is a row of 16 points along x, N the 16 output channels and
// K = 2 taps x 16 input channels per v_mfma_f32_16x16x32_bf16.  A workgroup
// computes a 16 x 8 x 4 block of points from an LDS copy of its input block
// plus a one-point margin.  The backward pass with respect to the input is the
// same kernel with flipped, transposed weights and a ReLU mask; the weight
// gradient is a second implicit GEMM on the matrix cores (K = points), its
// per-workgroup FP32 partials reduced in FP64 in a fixed order.  The training
// residual, its mean square and the augmentation by cube symmetries are
// kernels here too, so a training step is library calls only.
#include "kernels.h"

namespace gpm {

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int CV_TX = 16, CV_TY = 8, CV_TZ = 4, CV_NT = 256;
constexpr int CV_HX = CV_TX + 2, CV_HY = CV_TY + 2, CV_HZ = CV_TZ + 2;
constexpr int CV_HP = CV_HX * CV_HY * CV_HZ;  // halo points
constexpr int CV_KSTEPS = 14;                 // ceil(27 taps / 2)

__device__ __forceinline__ int tap_dz(int t) { return t / 9 - 1; }
__device__ __forceinline__ int tap_dy(int t) { return (t / 3) % 3 - 1; }
__device__ __forceinline__ int tap_dx(int t) { return t % 3 - 1; }

// 16 bytes a lane from global memory straight into LDS: lane l's go to lds + l (lds is the wave's, not the lane's);
// the wave's s_waitcnt vmcnt(0) tells that they are there
__device__ __forceinline__ void load_lds16(const uint16_t* g, uint4* lds) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)g,
                                   (__attribute__((address_space(3))) void*)lds, 16, 0, 0);
}

// mode: 0 = relu(conv + bias) -> bf16 [p][16]; 1 = (conv + bias)[0..2] * scale -> FP32 SoA [3][n^3];
//       2 = conv * (mask > 0) -> bf16 [p][16] (input gradient through a ReLU)
//
// The input block plus margin goes from global memory straight into LDS ([hz][hy][hx][16], 16 bytes a lane, all nine
// loads of a wave in flight; through registers one after the other they were most of the kernel's time).  The weights
// are the product's rows and the points its columns, so that a lane ends with 4 consecutive channels of one point
// and a row of 16 points is stored as 512 consecutive bytes.  A K-step holds two consecutive taps, the second in
// the upper lanes: it lies one point, one row or one plane further, so three lane addresses and immediate offsets
// reach all 27 taps of every row.
template <int MODE>
__global__ __launch_bounds__(CV_NT) void conv16_kernel(const uint16_t* __restrict__ in, const uint16_t* __restrict__ w,
                                                       const float* __restrict__ bias, int n, void* out,
                                                       const uint16_t* __restrict__ mask, const float* scale_ptr) {
  __shared__ uint4 tile[CV_HP * 2];
  const int x0 = blockIdx.x * CV_TX, y0 = blockIdx.y * CV_TY, z0 = blockIdx.z * CV_TZ;
  const long nn = (long)n * n;
  const int m = n - 1, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  constexpr int NLD = (CV_HP * 2 + CV_NT - 1) / CV_NT;
#pragma unroll
  for (int k = 0; k < NLD; ++k) {
    const int q0 = (wave + k * (CV_NT / 64)) * 64, q = q0 + lane;
    if (q < CV_HP * 2) {
      const int pt = q >> 1, half = q & 1;
      const int hx = pt % CV_HX, hy = (pt / CV_HX) % CV_HY, hz = pt / (CV_HX * CV_HY);
      const long g = (long)((z0 - 1 + hz) & m) * nn + (long)((y0 - 1 + hy) & m) * n + ((x0 - 1 + hx) & m);
      load_lds16(in + g * 16 + half * 8, tile + q0);
    }
  }
  const int col = lane & 15, grp = lane >> 4;
  // weight fragments ([tap][out][in] bfloat16, lane: out channel col, 8 input channels) of the 14 K-steps in registers
  v8bf wfrag[CV_KSTEPS];
#pragma unroll
  for (int s = 0; s < CV_KSTEPS; ++s) {
    const int t = 2 * s + (grp >> 1);
    uint4 u = make_uint4(0, 0, 0, 0);
    if (t < 27) u = *reinterpret_cast<const uint4*>(w + ((t * 16 + col) * 16 + 8 * (grp & 1)));
    wfrag[s] = __builtin_bit_cast(v8bf, u);
  }
  const float scale = (MODE == 1 && scale_ptr) ? scale_ptr[0] : 1.0f;
  float bco[4] = {0.f, 0.f, 0.f, 0.f};
  if (bias) {
#pragma unroll
    for (int j = 0; j < 4; ++j) bco[j] = bias[4 * grp + j];
  }
  const long n3 = nn * n;
  // each wave computes 8 rows of 16 points (one plane of the block)
  static_assert(CV_NT / 64 == CV_TZ, "one wave per plane");
  const int lz = wave;
  const int up = grp >> 1;
  const uint4* b0 = tile + (lz * CV_HY * CV_HX + col) * 2 + (grp & 1);  // point col of the plane's first row
  const uint4* b1 = b0 + up * 2;                                        // the second tap at the next point,
  const uint4* b2 = b0 + up * ((CV_HX - 2) * 2);                        // in the next row,
  const uint4* b3 = b0 + up * ((CV_HY * CV_HX - 2 * CV_HX - 2) * 2);    // in the next plane
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wave's part of the block is in LDS
  __syncthreads();
#pragma unroll
  for (int ly = 0; ly < CV_TY; ++ly) {
    v4f acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < CV_KSTEPS; ++s) {
      // (the 28th tap counts as zeros, not as the 27th's values under weight zero: those may be infinite)
      const int t = 2 * s, o = ((t / 9 * CV_HY + (t / 3) % 3 + ly) * CV_HX + t % 3) * 2;
      const uint4* b = (s == CV_KSTEPS - 1) ? b0 : (t % 3 != 2 ? b1 : ((t / 3) % 3 != 2 ? b2 : b3));
      uint4 v = b[o];
      if (s == CV_KSTEPS - 1 && up) v = make_uint4(0u, 0u, 0u, 0u);
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wfrag[s], __builtin_bit_cast(v8bf, v), acc, 0, 0, 0);
    }
    // D: lane holds output channels 4 grp + j of point col
    const long p = ((long)(z0 + lz) * n + (y0 + ly)) * n + (x0 + col);
    if constexpr (MODE == 1) {
      if (grp == 0) {
#pragma unroll
        for (int j = 0; j < 3; ++j) reinterpret_cast<float*>(out)[j * n3 + p] = (acc[j] + bco[j]) * scale;
      }
    } else {
      uint16_t r[4];
      if constexpr (MODE == 0) {
#pragma unroll
        for (int j = 0; j < 4; ++j) r[j] = f2bf(fmaxf(acc[j] + bco[j], 0.0f));
      } else {
        const uint2 mk = *reinterpret_cast<const uint2*>(mask + p * 16 + 4 * grp);
        const uint16_t mw[4] = {(uint16_t)mk.x, (uint16_t)(mk.x >> 16), (uint16_t)mk.y, (uint16_t)(mk.y >> 16)};
#pragma unroll
        for (int j = 0; j < 4; ++j) r[j] = f2bf(bf2f(mw[j]) > 0.0f ? acc[j] : 0.0f);
      }
      *reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(out) + p * 16 + 4 * grp) =
          make_uint2((uint32_t)r[0] | ((uint32_t)r[1] << 16), (uint32_t)r[2] | ((uint32_t)r[3] << 16));
    }
  }
}

// Weight gradient of one layer on the matrix cores: for each tap t,
// dW_t[co][ci] = sum_p dy[p][co] x[p + d_t][ci] is a 16 x 16 GEMM with K running over the
// points.  One MFMA takes 32 points (two x-rows of a 16 x 8 x 4 tile): A[co][k] = dy[p_k][co],
// B[k][ci] = x[p_k + d_t][ci].  Both operands need 8 consecutive points per lane for one channel, the transpose of
// the [point][16] layout in memory: the tile goes straight into LDS as it is (16 bytes a lane) and is transposed by
// the reads (ds_read_b64_tr_b16: of the 4 points x 16 channels that the addresses of 16 lanes cover, lane i gets
// channel i of the 4 points), so that a tap's shift is an address.  (Transposed into LDS by 2-byte stores the kernel
// took 137 us at 128^3 and 1.04 ms at 256^3.)  Wave w owns taps w, w + 4, ..., and wave 3's spare slot accumulates the
// bias gradient (B = ones).  A workgroup walks tiles blockIdx.x, + gridDim.x, ... and writes
// one FP32 partial; the partials are summed in a fixed order in FP64.
constexpr int WG_PART = 27 * 256 + 16;                  // one partial: [t][co][ci] then the bias [co]
constexpr int WG_GRID = 768;                            // workgroups (partials) at most: 3 a CU (51 KB of LDS each)

typedef short v4s __attribute__((ext_vector_type(4)));
typedef short v8s __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) v4s lds_v4s;

// channel lane % 16 of the 8 points from byte offset `at` of p on (this lane's part of the first four; the next four
// are 128 bytes further)
__device__ __forceinline__ v8bf read_points8(const uint8_t* p, int at) {
  const v4s a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s*)(p + at));
  const v4s b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s*)(p + at + 128));
  return __builtin_bit_cast(v8bf, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
}

__global__ __launch_bounds__(CV_NT) void conv16_wgrad_kernel(const uint16_t* __restrict__ x,
                                                             const uint16_t* __restrict__ dy, int n, long ntiles,
                                                             float* __restrict__ part) {
  __shared__ uint4 xt[CV_HP * 2];                  // [hz][hy][hx][16]
  __shared__ uint4 dyt[CV_TX * CV_TY * CV_TZ * 2]; // [lz][ly][lx][16]
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int col = lane & 15, grp = lane >> 4;
  const int ntx = n / CV_TX, nty = n / CV_TY;
  const int m = n - 1;
  const long nn = (long)n * n;
  v4f acc[7];
#pragma unroll
  for (int j = 0; j < 7; ++j) acc[j] = v4f{0.f, 0.f, 0.f, 0.f};
  const v8bf ones = __builtin_bit_cast(v8bf, make_uint4(0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u));
  // lane's read addresses: points 8 (grp & 1) + (lane % 16) / 4 of x-row grp / 2 of a pair, 4 channels each
  const int px = 8 * (grp & 1) + (col >> 2), pr = grp >> 1;
  const uint8_t* ab = reinterpret_cast<const uint8_t*>(dyt) + (pr * CV_TX + px) * 32 + (col & 3) * 8;
  const uint8_t* xb[7];
#pragma unroll
  for (int j = 0; j < 7; ++j) {
    const int t = min(wave + 4 * j, 26);
    const int off = ((1 + tap_dz(t)) * CV_HY + 1 + tap_dy(t)) * CV_HX + 1 + tap_dx(t);
    xb[j] = reinterpret_cast<const uint8_t*>(xt) + (off + pr * CV_HX + px) * 32 + (col & 3) * 8;
  }
  for (long tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const int x0 = (int)(tile % ntx) * CV_TX, y0 = (int)((tile / ntx) % nty) * CV_TY;
    const int z0 = (int)(tile / ((long)ntx * nty)) * CV_TZ;
    __syncthreads();  // the previous tile's operands are consumed
    constexpr int NX = (CV_HP * 2 + CV_NT - 1) / CV_NT, ND = CV_TX * CV_TY * CV_TZ * 2 / CV_NT;
#pragma unroll
    for (int k = 0; k < NX; ++k) {
      const int q0 = (wave + k * (CV_NT / 64)) * 64, q = q0 + lane;
      if (q < CV_HP * 2) {
        const int pt = q >> 1, half = q & 1;
        const int hx = pt % CV_HX, hy = (pt / CV_HX) % CV_HY, hz = pt / (CV_HX * CV_HY);
        const long g = (long)((z0 - 1 + hz) & m) * nn + (long)((y0 - 1 + hy) & m) * n + ((x0 - 1 + hx) & m);
        load_lds16(x + g * 16 + half * 8, xt + q0);
      }
    }
#pragma unroll
    for (int k = 0; k < ND; ++k) {
      const int q0 = (wave + k * (CV_NT / 64)) * 64, q = q0 + lane;
      const int pt = q >> 1, half = q & 1;
      const int lx = pt % CV_TX, row = pt / CV_TX;  // row = ly + 8 lz
      const long g = ((long)(z0 + row / CV_TY) * n + (y0 + row % CV_TY)) * n + (x0 + lx);
      load_lds16(dy + g * 16 + half * 8, dyt + q0);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wave's part of the tile is in LDS
    __syncthreads();
    // K-step s: points lx = 8 (grp & 1) + e, e < 8, of row 2 s + (grp >> 1)
#pragma unroll
    for (int s = 0; s < CV_TY * CV_TZ / 2; ++s) {
      const v8bf a = read_points8(ab, s * 2 * CV_TX * 32);
      const int xo = ((2 * s / CV_TY) * CV_HY + 2 * s % CV_TY) * CV_HX * 32;
#pragma unroll
      for (int j = 0; j < 7; ++j) {
        const bool bias_slot = j == 6 && wave == 3;
        const v8bf b = bias_slot ? ones : read_points8(xb[j], xo);
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc[j], 0, 0, 0);
      }
    }
  }
  // D: lane holds co = 4 grp + r of column ci = col
  float* o = part + (long)blockIdx.x * WG_PART;
#pragma unroll
  for (int j = 0; j < 7; ++j) {
    const int t = wave + 4 * j;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int co = 4 * grp + r;
      if (t < 27) o[(t * 16 + co) * 16 + col] = acc[j][r];
      else if (col == 0) o[27 * 256 + co] = acc[j][r];
    }
  }
}

// sum the partials in a fixed order (FP64) and scatter into the flat parameter-gradient layout
// W[co][ci][27] b[co] of layer (ci_n -> co_n) at offset off; 64 entries per workgroup, each of 16 waves
// adds a contiguous sixteenth of the partials (four sixteenths took 34 us, a latency chain of 128 loads) and
// the parts are combined in order
constexpr int WR_PARTS = 16;
__global__ __launch_bounds__(64 * WR_PARTS) void wgrad_reduce_kernel(const float* __restrict__ part, int nblk, int ci_n,
                                                                     int co_n, float* __restrict__ grad, long off) {
  __shared__ double q[WR_PARTS][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int e = blockIdx.x * 64 + lane;
  const int lo = wave * nblk / WR_PARTS, hi = (wave + 1) * nblk / WR_PARTS;
  double s = 0.0;
  if (e < WG_PART) {
#pragma unroll 8
    for (int b = lo; b < hi; ++b) s += (double)part[(long)b * WG_PART + e];
  }
  q[wave][lane] = s;
  __syncthreads();
  if (wave != 0 || e >= WG_PART) return;
  s = q[0][lane];
#pragma unroll
  for (int w = 1; w < WR_PARTS; ++w) s += q[w][lane];
  if (e < 27 * 256) {
    const int t = e / 256, co = (e / 16) % 16, ci = e % 16;
    if (co < co_n && ci < ci_n) grad[off + ((long)co * ci_n + ci) * 27 + t] = (float)s;
  } else {
    const int co = e - 27 * 256;
    if (co < co_n) grad[off + (long)co_n * ci_n * 27 + co] = (float)s;
  }
}

// flat FP32 parameters -> bf16 forward weights [L][t][co][ci], backward-data weights
// [L][t'][ci][co] (t' = 26 - t), FP32 biases [L][16]; padded channels are zero
__global__ __launch_bounds__(256) void pack_weights_kernel(const float* __restrict__ p, uint16_t* wf, uint16_t* wb,
                                                           float* bias) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;  // over 3 * 27 * 256
  const int cis[3] = {4, 16, 16}, cos_[3] = {16, 16, 3};
  const long offs[3] = {0, 16 * 4 * 27 + 16, 16 * 4 * 27 + 16 + 16 * 16 * 27 + 16};
  if (e < 3 * 16) {
    const int L = e / 16, co = e % 16;
    bias[e] = co < cos_[L] ? p[offs[L] + (long)cos_[L] * cis[L] * 27 + co] : 0.f;
  }
  if (e >= 3 * 27 * 256) return;
  const int L = e / (27 * 256), r = e % (27 * 256);
  const int t = r / 256, a = (r / 16) % 16, b = r % 16;
  // forward: wf[L][t][co = a][ci = b]
  float vf = 0.f;
  if (a < cos_[L] && b < cis[L]) vf = p[offs[L] + ((long)a * cis[L] + b) * 27 + t];
  wf[e] = f2bf(vf);
  // backward data: wb[L][t][ci = a][co = b] = W[co][ci][26 - t]
  float vb = 0.f;
  if (b < cos_[L] && a < cis[L]) vb = p[offs[L] + ((long)b * cis[L] + a) * 27 + (26 - t)];
  wb[e] = f2bf(vb);
}

// Adam on the FP32 master parameters (bias-corrected)
// (1 - beta) is passed separately: forming it in FP32 from beta = 0.999f would cost 5e-5 relative
__global__ __launch_bounds__(256) void adam_kernel(float* p, float* m, float* v, const float* g, int np, float lr,
                                                   float b1, float b2, float omb1, float omb2, float eps, float c1,
                                                   float c2) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= np) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + omb1 * gi;
  const float vi = b2 * v[i] + omb2 * gi * gi;
  m[i] = mi;
  v[i] = vi;
  p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

// ---------------------------------------------------------------------------
// inputs: channel 0 = sign(delta) log(1 + |delta|), channels 1..3 = grad phi / rms|grad phi|
// ---------------------------------------------------------------------------
// One pass over both inputs: FP64 partials of |grad phi|^2 (part[0 .. blocks)) and of n00 (part[blocks .. 2 blocks)).
// Four consecutive x a thread; a grid of whole rounds of the chip in place of 512 workgroups with two 64-bit
// divisions a point (100 us, and 55 us for the separate sum of n00, at 256^3).
constexpr int FEAT_BLOCKS = 2048;
template <typename T>
__global__ __launch_bounds__(256) void field_sums_kernel(const T* __restrict__ n00, const T* __restrict__ phi, int lg,
                                                         double* part) {
  __shared__ double red[2][4];
  const int n = 1 << lg, m = n - 1;
  const long nn = 1L << (2 * lg), n4 = nn << lg >> 2;
  const double hn = 0.5 * n;
  double g2 = 0.0, s0 = 0.0;
  for (long q = (long)blockIdx.x * 256 + threadIdx.x; q < n4; q += (long)gridDim.x * 256) {
    const long i = q * 4;
    const int x = (int)i & m, y = (int)(i >> lg) & m, z = (int)(i >> (2 * lg));
    const long row = i - x;
    const V4<T> c = *reinterpret_cast<const V4<T>*>(phi + i);
    const T xm = phi[row + ((x - 1) & m)], xp = phi[row + ((x + 4) & m)];
    const long rz = (long)z << (2 * lg), ry = (long)y << lg;
    const V4<T> yp = *reinterpret_cast<const V4<T>*>(phi + rz + ((long)((y + 1) & m) << lg) + x);
    const V4<T> ym = *reinterpret_cast<const V4<T>*>(phi + rz + ((long)((y - 1) & m) << lg) + x);
    const V4<T> zp = *reinterpret_cast<const V4<T>*>(phi + ((long)((z + 1) & m) << (2 * lg)) + ry + x);
    const V4<T> zm = *reinterpret_cast<const V4<T>*>(phi + ((long)((z - 1) & m) << (2 * lg)) + ry + x);
    const V4<T> d = *reinterpret_cast<const V4<T>*>(n00 + i);
    auto add = [&](T a, T b) {
      const double g = ((double)a - (double)b) * hn;
      g2 += g * g;
    };
    add(c.y, xm); add(c.z, c.x); add(c.w, c.y); add(xp, c.z);
    add(yp.x, ym.x); add(yp.y, ym.y); add(yp.z, ym.z); add(yp.w, ym.w);
    add(zp.x, zm.x); add(zp.y, zm.y); add(zp.z, zm.z); add(zp.w, zm.w);
    s0 += ((double)d.x + (double)d.y) + ((double)d.z + (double)d.w);
  }
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) {
    g2 += __shfl_down(g2, d);
    s0 += __shfl_down(s0, d);
  }
  if ((threadIdx.x & 63) == 0) {
    red[0][threadIdx.x >> 6] = g2;
    red[1][threadIdx.x >> 6] = s0;
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    const double* r = red[threadIdx.x];
    part[threadIdx.x * gridDim.x + blockIdx.x] = ((r[0] + r[1]) + r[2]) + r[3];
  }
}

// rms |grad phi| (FP32) and the sum of n00 from the partials
__global__ __launch_bounds__(256) void field_sums_final_kernel(const double* part, int nb, long n3, float* rms,
                                                               double* n00_sum) {
  __shared__ double red[2][256];
  double g = 0.0, s = 0.0;
  for (int i = threadIdx.x; i < nb; i += 256) {
    g += part[i];
    s += part[nb + i];
  }
  red[0][threadIdx.x] = g;
  red[1][threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) {
      red[0][threadIdx.x] += red[0][threadIdx.x + w];
      red[1][threadIdx.x] += red[1][threadIdx.x + w];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    rms[0] = (float)sqrt(red[0][0] / (double)n3);
    n00_sum[0] = red[1][0];
  }
}

// two threads a point, each storing half of its 32 bytes (channels 4 .. 15 are zero)
template <typename T>
__global__ __launch_bounds__(256) void features_kernel(const T* __restrict__ n00, const T* __restrict__ phi, int lg,
                                                       const double* __restrict__ n00_sum, const float* __restrict__ rms,
                                                       uint16_t* __restrict__ out) {
  const int n = 1 << lg, m = n - 1;
  const long q = (long)blockIdx.x * 256 + threadIdx.x, i = q >> 1;  // the grid is exact: 2 n^3 is a multiple of 256
  uint4 a = make_uint4(0u, 0u, 0u, 0u);
  if ((q & 1) == 0) {
    const int x = (int)i & m, y = (int)(i >> lg) & m, z = (int)(i >> (2 * lg));
    const long rz = (long)z << (2 * lg), ry = (long)y << lg;
    const float hn = 0.5f * n;
    const float mean = (float)(n00_sum[0] / (double)(1L << (3 * lg)));
    const float delta = (float)n00[i] / mean - 1.0f;
    const float s = copysignf(log1pf(fabsf(delta)), delta);
    const float ir = 1.0f / rms[0];
    const float gx = (float)(phi[rz + ry + ((x + 1) & m)] - phi[rz + ry + ((x - 1) & m)]) * hn * ir;
    const float gy = (float)(phi[rz + ((long)((y + 1) & m) << lg) + x] - phi[rz + ((long)((y - 1) & m) << lg) + x]) * hn * ir;
    const float gz = (float)(phi[((long)((z + 1) & m) << (2 * lg)) + ry + x] -
                             phi[((long)((z - 1) & m) << (2 * lg)) + ry + x]) * hn * ir;
    a.x = (uint32_t)f2bf(s) | ((uint32_t)f2bf(gx) << 16);
    a.y = (uint32_t)f2bf(gy) | ((uint32_t)f2bf(gz) << 16);
  }
  reinterpret_cast<uint4*>(out)[q] = a;
}

// ---------------------------------------------------------------------------
// particle-side helpers: CIC gather of a 3-component FP32 SoA field
// ---------------------------------------------------------------------------
__device__ __forceinline__ void cic(double x, int n, int& i0, int& i1, float& w0, float& w1) {
  const double s = x * (double)n;
  const double fl = floor(s);
  const float f = (float)(s - fl);
  i0 = ((int)fl) & (n - 1);
  i1 = (i0 + 1) & (n - 1);
  w0 = 1.0f - f;
  w1 = f;
}

// CIC interpolation of the 3-component FP32 SoA field f at particle i
template <typename T>
__device__ __forceinline__ void gather3_at(const Particles<T>& p, long i, int n, const float* __restrict__ f,
                                           float v[3]) {
  int x0, x1, y0, y1, z0, z1;
  float wx0, wx1, wy0, wy1, wz0, wz1;
  Particle<T> q;
  load_pos(p, i, q);
  cic(q.x, n, x0, x1, wx0, wx1);
  cic(q.y, n, y0, y1, wy0, wy1);
  cic(q.z, n, z0, z1, wz0, wz1);
  const long nn = (long)n * n, n3 = nn * n;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const float* g = f + c * n3;
    v[c] = wz0 * (wy0 * (wx0 * g[z0 * nn + y0 * n + x0] + wx1 * g[z0 * nn + y0 * n + x1]) +
                  wy1 * (wx0 * g[z0 * nn + y1 * n + x0] + wx1 * g[z0 * nn + y1 * n + x1])) +
           wz1 * (wy0 * (wx0 * g[z1 * nn + y0 * n + x0] + wx1 * g[z1 * nn + y0 * n + x1]) +
                  wy1 * (wx0 * g[z1 * nn + y1 * n + x0] + wx1 * g[z1 * nn + y1 * n + x1]));
  }
}

template <typename T>
__global__ __launch_bounds__(256) void gather3_kernel(Particles<T> p, long np, int n, const float* __restrict__ f,
                                                      float* __restrict__ out) {
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i >= np) return;
  float v[3];
  gather3_at(p, i, n, f, v);
  *reinterpret_cast<V3<float>*>(out + 3 * (long)load_id(p, i)) = V3<float>{v[0], v[1], v[2]};
}

// Training residual: pred = gathered network output, r = pred - target (FP32, identifier order),
// dpred = gscale r, and FP64 per-workgroup sums of |r|^2 and |target|^2 (fixed grid, fixed order).
constexpr int LOSS_BLOCKS = 512;
template <typename T>
__global__ __launch_bounds__(256) void loss3_kernel(Particles<T> p, long np, int n, const float* __restrict__ f,
                                                    const float* __restrict__ target, float gscale,
                                                    float* __restrict__ dpred, double* __restrict__ part) {
  __shared__ double red[2][256];
  double e2 = 0.0, t2 = 0.0;
  for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < np; i += (long)gridDim.x * 256) {
    float v[3];
    gather3_at(p, i, n, f, v);
    const long id = load_id(p, i);
    const V3<float> t3 = *reinterpret_cast<const V3<float>*>(target + 3 * id);
    const float tg[3] = {t3.x, t3.y, t3.z};
    float d[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const float r = v[c] - tg[c];
      d[c] = r * gscale;
      e2 += (double)r * (double)r;
      t2 += (double)tg[c] * (double)tg[c];
    }
    *reinterpret_cast<V3<float>*>(dpred + 3 * id) = V3<float>{d[0], d[1], d[2]};
  }
  red[0][threadIdx.x] = e2;
  red[1][threadIdx.x] = t2;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) {
      red[0][threadIdx.x] += red[0][threadIdx.x + s];
      red[1][threadIdx.x] += red[1][threadIdx.x + s];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    part[2 * blockIdx.x] = red[0][0];
    part[2 * blockIdx.x + 1] = red[1][0];
  }
}

// out[0] = mean |r|^2, out[1] = mean |target|^2 over the 3 np components
__global__ __launch_bounds__(256) void loss3_final_kernel(const double* __restrict__ part, int nb, double inv_count,
                                                          double* __restrict__ out) {
  __shared__ double red[2][256];
  double e2 = 0.0, t2 = 0.0;
  for (int b = threadIdx.x; b < nb; b += 256) {
    e2 += part[2 * b];
    t2 += part[2 * b + 1];
  }
  red[0][threadIdx.x] = e2;
  red[1][threadIdx.x] = t2;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) {
      red[0][threadIdx.x] += red[0][threadIdx.x + s];
      red[1][threadIdx.x] += red[1][threadIdx.x + s];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    out[0] = red[0][0] * inv_count;
    out[1] = red[1][0] * inv_count;
  }
}

// One of the 48 symmetries of the periodic unit cube on particle data: component d of the result
// is component perm[d] of the input, reflected (x -> 1 - x, wrapped into [0, 1)) for positions and
// negated for the two vector fields where flip bit d is set.  Each thread reads its particle before
// writing it, so the outputs may alias the inputs.
__global__ __launch_bounds__(256) void cube_symmetry_kernel(long np, int p0, int p1, int p2, int flip,
                                                            const double* pos, const float* u, const float* v,
                                                            double* pos_out, float* u_out, float* v_out) {
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i >= np) return;
  const int perm[3] = {p0, p1, p2};
  double x[3];
  float a[3], b[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    x[d] = pos[3 * i + perm[d]];
    a[d] = u[3 * i + perm[d]];
    b[d] = v[3 * i + perm[d]];
  }
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const bool f = (flip >> d) & 1;
    double y = x[d];
    if (f) {
      y = 1.0 - y;
      if (y >= 1.0) y -= 1.0;
    }
    pos_out[3 * i + d] = y;
    u_out[3 * i + d] = f ? -a[d] : a[d];
    v_out[3 * i + d] = f ? -b[d] : b[d];
  }
}

// gradient of phi (centred differences, CIC-interpolated) at the particles, identifier order
template <typename T>
__global__ __launch_bounds__(256) void gather_grad_phi_kernel(Particles<T> p, long np, int n, const T* __restrict__ phi,
                                                              T* __restrict__ out) {
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i >= np) return;
  const int m = n - 1;
  const long nn = (long)n * n;
  int ix[2], iy[2], iz[2];
  T wx[2], wy[2], wz[2];
  {
    Particle<T> q;
    load_pos(p, i, q);
    const double sx = q.x * (double)n, sy = q.y * (double)n, sz = q.z * (double)n;
    const double fx = floor(sx), fy = floor(sy), fz = floor(sz);
    ix[0] = ((int)fx) & m; iy[0] = ((int)fy) & m; iz[0] = ((int)fz) & m;
    ix[1] = (ix[0] + 1) & m; iy[1] = (iy[0] + 1) & m; iz[1] = (iz[0] + 1) & m;
    wx[1] = (T)(sx - fx); wy[1] = (T)(sy - fy); wz[1] = (T)(sz - fz);
    wx[0] = (T)1 - wx[1]; wy[0] = (T)1 - wy[1]; wz[0] = (T)1 - wz[1];
  }
  T g[3] = {0, 0, 0};
  for (int a = 0; a < 2; ++a)
    for (int b = 0; b < 2; ++b)
      for (int c = 0; c < 2; ++c) {
        const int z = iz[a], y = iy[b], x = ix[c];
        const T w = wz[a] * wy[b] * wx[c];
        g[0] += w * (phi[z * nn + y * n + ((x + 1) & m)] - phi[z * nn + y * n + ((x - 1) & m)]);
        g[1] += w * (phi[z * nn + ((y + 1) & m) * n + x] - phi[z * nn + ((y - 1) & m) * n + x]);
        g[2] += w * (phi[((z + 1) & m) * nn + y * n + x] - phi[((z - 1) & m) * nn + y * n + x]);
      }
  const T hn = (T)(0.5 * n);
  *reinterpret_cast<V3<T>*>(out + 3 * (long)load_id(p, i)) = V3<T>{g[0] * hn, g[1] * hn, g[2] * hn};
}

// ---------------------------------------------------------------------------
// host launchers
// ---------------------------------------------------------------------------
void closure_pack(const float* params, uint16_t* wf, uint16_t* wb, float* bias, hipStream_t st) {
  hipLaunchKernelGGL(pack_weights_kernel, dim3((3 * 27 * 256 + 255) / 256), dim3(256), 0, st, params, wf, wb, bias);
}

void closure_conv(const uint16_t* in, const uint16_t* w, const float* bias, int n, int mode, void* out,
                  const uint16_t* mask, const float* scale, hipStream_t st) {
  dim3 grid(n / CV_TX, n / CV_TY, n / CV_TZ);
  if (mode == 0)
    hipLaunchKernelGGL((conv16_kernel<0>), grid, dim3(CV_NT), 0, st, in, w, bias, n, out, mask, scale);
  else if (mode == 1)
    hipLaunchKernelGGL((conv16_kernel<1>), grid, dim3(CV_NT), 0, st, in, w, bias, n, out, mask, scale);
  else
    hipLaunchKernelGGL((conv16_kernel<2>), grid, dim3(CV_NT), 0, st, in, w, bias, n, out, mask, scale);
}

static long closure_wgrad_tiles(int n) { return (long)(n / CV_TX) * (n / CV_TY) * (n / CV_TZ); }
// workgroups of the weight-gradient kernel: every workgroup takes at least two tiles (so that the
// tile walk runs at every size), at most WG_GRID workgroups
static int closure_wgrad_grid(int n) {
  const long h = closure_wgrad_tiles(n) / 2;
  return (int)(h < 1 ? 1 : (h < WG_GRID ? h : WG_GRID));
}
long closure_wgrad_part_bytes(int n) { return (long)closure_wgrad_grid(n) * WG_PART * 4; }

void closure_wgrad(const uint16_t* x, const uint16_t* dy, int n, float* part, int ci_n, int co_n, float* grad,
                   long off, hipStream_t st) {
  const long tiles = closure_wgrad_tiles(n);
  const int grid = closure_wgrad_grid(n);
  hipLaunchKernelGGL(conv16_wgrad_kernel, dim3(grid), dim3(CV_NT), 0, st, x, dy, n, tiles, part);
  hipLaunchKernelGGL(wgrad_reduce_kernel, dim3((WG_PART + 63) / 64), dim3(64 * WR_PARTS), 0, st, part, grid, ci_n, co_n, grad,
                     off);
}

void closure_adam(float* p, float* m, float* v, const float* g, int np, double lr, int step, hipStream_t st) {
  const double b1 = 0.9, b2 = 0.999;
  const float c1 = (float)(1.0 - pow(b1, step)), c2 = (float)(1.0 - pow(b2, step));
  hipLaunchKernelGGL(adam_kernel, dim3((np + 255) / 256), dim3(256), 0, st, p, m, v, g, np, (float)lr, (float)b1,
                     (float)b2, (float)(1.0 - b1), (float)(1.0 - b2), 1e-8f, c1, c2);
}

template <typename T>
void closure_features(const T* n00, const T* phi, int n, double* n00_sum, double* part, float* rms, uint16_t* out,
                      hipStream_t st) {
  const long n3 = (long)n * n * n;
  int lg = 0;
  while ((1 << lg) < n) ++lg;
  const long want = (n3 / 4 + 255) / 256;
  const int nb = (int)(want < FEAT_BLOCKS ? want : FEAT_BLOCKS);
  hipLaunchKernelGGL((field_sums_kernel<T>), dim3(nb), dim3(256), 0, st, n00, phi, lg, part);
  hipLaunchKernelGGL(field_sums_final_kernel, dim3(1), dim3(256), 0, st, part, nb, n3, rms, n00_sum);
  hipLaunchKernelGGL((features_kernel<T>), dim3((unsigned)(2 * n3 / 256)), dim3(256), 0, st, n00, phi, lg, n00_sum, rms,
                     out);
}

template <typename T>
void closure_gather3(const Particles<T>& p, long np, int n, const float* f, float* out, hipStream_t st) {
  hipLaunchKernelGGL((gather3_kernel<T>), dim3((unsigned)((np + 255) / 256)), dim3(256), 0, st, p, np, n, f, out);
}

template <typename T>
void closure_loss3(const Particles<T>& p, long np, int n, const float* f, const float* target, float* dpred,
                   double* part, double* out, hipStream_t st) {
  const long want = (np + 255) / 256;
  const int nb = (int)(want < LOSS_BLOCKS ? (want > 0 ? want : 1) : LOSS_BLOCKS);
  const float gscale = (float)(2.0 / (3.0 * (double)np));
  hipLaunchKernelGGL((loss3_kernel<T>), dim3(nb), dim3(256), 0, st, p, np, n, f, target, gscale, dpred, part);
  hipLaunchKernelGGL(loss3_final_kernel, dim3(1), dim3(256), 0, st, part, nb, 1.0 / (3.0 * (double)np), out);
}

void closure_cube_symmetry(long np, const int perm[3], int flip, const double* pos, const float* u, const float* v,
                           double* pos_out, float* u_out, float* v_out, hipStream_t st) {
  hipLaunchKernelGGL(cube_symmetry_kernel, dim3((unsigned)((np + 255) / 256)), dim3(256), 0, st, np, perm[0], perm[1],
                     perm[2], flip, pos, u, v, pos_out, u_out, v_out);
}

template <typename T>
void gather_grad_phi(const Particles<T>& p, long np, int n, const T* phi, T* out, hipStream_t st) {
  hipLaunchKernelGGL((gather_grad_phi_kernel<T>), dim3((unsigned)((np + 255) / 256)), dim3(256), 0, st, p, np, n, phi,
                     out);
}

#define GPM_CL_INST(T)                                                                                          \
  template void closure_features<T>(const T*, const T*, int, double*, double*, float*, uint16_t*, hipStream_t);   \
  template void closure_gather3<T>(const Particles<T>&, long, int, const float*, float*, hipStream_t);          \
  template void closure_loss3<T>(const Particles<T>&, long, int, const float*, const float*, float*, double*,     \
                                 double*, hipStream_t);                                                          \
  template void gather_grad_phi<T>(const Particles<T>&, long, int, const T*, T*, hipStream_t);
GPM_CL_INST(float)
GPM_CL_INST(double)

}  // namespace gpm
