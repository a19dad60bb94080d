// Training the two-layer perceptron of Sec. 2.1 (Eqns. 5-6) on encodings
// with known normal flows.  The paper delegates its loss and sampling to its
// predecessor; the loss here is our own: the mean over rows of the squared
// error of the predicted 2-vector,
//   L = (1/M) sum_r ||W2 relu(W1 x_r + b1) + b2 - y_r||^2,
// with the chain-rule gradients
//   dp_r = 2 (p_r - y_r) / M,  dW2 = sum_r dp_r h_r^T,  db2 = sum_r dp_r,
//   dz_r = (W2^T dp_r) * [z_r > 0],  dW1 = sum_r dz_r x_r^T,  db1 = sum_r dz_r,
// then plain gradient descent or Adam.  Every value is fp32; every reduction
// over rows runs in a fixed order (per-block partial sums, then a fixed tree
// over blocks), so a step is deterministic.
//
// Three launches per step:
//   k_train_fwd  layer 1, layer 2, the loss and the way back to dz; the
//                activations never leave the registers
//   k_train_dw1  dW1 = dZ^T X, split over rows
//   k_train_end  the partial sums and the update
//
// Both contractions run on the bf16 matrix cores at fp32 accuracy: an fp32
// operand of ordinary size is the exact sum of three bf16 terms (h + m + l, 8
// bits each; the usual expansion of a number into non-overlapping parts), and
// the products hh, hm, mh, mm, hl, lh keep everything above 2^-26 of a
// product; sums are fp32.  Six bf16 products of a 32 x 32 x 16 tile take 192
// cycles of a SIMD's matrix core, the eight fp32 products of that tile 512.
// 900k rows, D = 128, 256 units: k_train_fwd 0.75 ms and k_train_dw1 0.78 ms
// (0.93 PFLOP/s of bf16 products; a large bf16 GEMM reaches 1.2 on this card),
// k_train_end 18 us, against 6.5 ms per step for fp32 vector-ALU GEMMs with H
// stored; the error against 64 bits is the same.
// A tile whose operands hold a value that three bf16 terms do not carry is
// computed again on the fp32 matrix cores, which treat it as fp32 arithmetic
// does: an infinity, a NaN, |v| >= 2^127 (h may round to infinity), or a value
// under 2^-110 whose last bits lie under bf16's smallest number, 2^-133, so that
// l would lose them (both matrix cores keep subnormal operands, products and
// sums).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "sync.h"
#include "veckm_internal.h"

namespace veckm {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr uint32_t kHuge = 0x7f000000u;  // 2^127
// What was seen of the values split so far: the largest magnitude (as bits), and
// the bits of the last remainders, whose lower half is zero where they are bf16
// numbers (the third term carries them whole).
struct Extent {
  uint32_t big = 0, rest = 0;
  __device__ inline void take(float v, float r2) {
    const uint32_t mag = __float_as_uint(v) & 0x7fffffffu;
    big = mag > big ? mag : big;
    rest |= __float_as_uint(r2);
  }
  __device__ inline bool beyond_terms() const { return big >= kHuge || (rest & 0xffffu) != 0; }
};

// The three bf16 terms of 8 fp32 values, and what was seen of those.
struct Split8 {
  bf16x8 t[3];
  __device__ inline void make(const float (&v)[8], Extent& ext) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const __bf16 h = (__bf16)v[e];
      const float r1 = v[e] - (float)h;
      const __bf16 m = (__bf16)r1;
      const float r2 = r1 - (float)m;
      t[0][e] = h;
      t[1][e] = m;
      t[2][e] = (__bf16)r2;
      ext.take(v[e], r2);
    }
  }
};

// acc += a b over the six leading products of the split operands, smallest first.
__device__ inline floatx16 mfma_split(const bf16x8 (&a)[3], const bf16x8 (&b)[3], floatx16 acc) {
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], b[2], acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[2], b[0], acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[1], b[1], acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], b[1], acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[1], b[0], acc, 0, 0, 0);
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], b[0], acc, 0, 0, 0);
}

// W1's fragments (the B operand of layer 1): per 16-feature k-step, 32-unit
// tile and bf16 term, lane l holds features 8 (l >> 5) + (0..7) of unit l & 31.
__device__ inline void put_w1_frag(uint16_t* frag, int nt, int hid, int k, float w, int* bad) {
  const __bf16 h = (__bf16)w;
  const float r1 = w - (float)h;
  const __bf16 m = (__bf16)r1;
  const float r2 = r1 - (float)m;
  const __bf16 t[3] = {h, m, (__bf16)r2};
  Extent ext;
  ext.take(w, r2);
  if (ext.beyond_terms()) *bad = 1;  // (stays set: layer 1 runs in fp32)
  const int lane = ((k >> 3) & 1) * 32 + (hid & 31);
  uint16_t* p = frag + (((int64_t)(k >> 4) * nt + (hid >> 5)) * 3 * 64 + lane) * 8 + (k & 7);
#pragma unroll
  for (int s = 0; s < 3; ++s) {
    uint16_t u;
    __builtin_memcpy(&u, &t[s], 2);
    p[s * 64 * 8] = u;
  }
}

__global__ void k_w1_frag(const float* __restrict__ W1, int k2, int hidden, int k2pad,
                          uint16_t* __restrict__ frag, int* __restrict__ bad) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= hidden * k2pad) return;
  const int hid = i / k2pad, k = i % k2pad;
  put_w1_frag(frag, hidden >> 5, hid, k, k < k2 ? W1[(int64_t)hid * k2 + k] : 0.f, bad);
}

// Sum over the 32 lanes of each half wave, in every lane.
__device__ inline float half_wave_sum(float v) {
  auto dpp = [](float x, auto ctrl) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), decltype(ctrl)::value,
                                                      0xf, 0xf, true));
  };
  v += dpp(v, std::integral_constant<int, 0xB1>{});   // lane ^ 1
  v += dpp(v, std::integral_constant<int, 0x4E>{});   // lane ^ 2
  v += dpp(v, std::integral_constant<int, 0x141>{});  // the other quad of 8
  v += dpp(v, std::integral_constant<int, 0x140>{});  // the other 8 of 16
  return v + __int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(v), 0x401F));  // lane ^ 16
}

struct FwdArgs {
  int64_t M;
  int k2, ksteps;
  int vec4;            // rows of x are 16-byte aligned
  const float* x;
  const float* y;
  const uint4* frag;   // W1's fragments
  const float* W1;
  const float* b1;
  const float* W2;
  const float* b2;
  const int* bad;      // W1 holds a value the bf16 terms cannot carry
  float inv_m;
  float* dZ;
  float* part;
};

// A wave takes 32 rows over every hidden unit (NT tiles of 32): rows are the
// M dimension, hidden units the N dimension, so a lane ends with 16 rows of
// unit l & 31 of each tile.  Sums over rows (db1, dW2) then stay in the lane,
// layer 2 is one reduction over 32 lanes for 16 rows at a time, and H is never
// stored.  The W1 slab of a k-step (NT x 3 KB) comes through LDS, shared by
// the block's waves and copied one step ahead; a lane reads its x row straight
// into the A operand (8 consecutive features), also one step ahead, across
// the ends of row blocks too.
//
// dZ goes out as the accumulators lie: [row tile of 32][unit tile][row octet]
// [lane][4], full 1 KB stores, zeros for the block's rows past M (dZ is sized
// in whole blocks); k_train_dw1 reads it as its A operand unchanged.  Per block the partial sums [db1 | dW2 (2) | db2
// (2) | loss] go to part[blockIdx.x], the parameter order after W1.
template <int NT, int NW>
__global__ __launch_bounds__(NW * 64) void k_train_fwd(FwdArgs a) {
  constexpr int HID = NT * 32, NP = 3 * HID + 3, SLAB = NT * 3 * 64;
  extern __shared__ __align__(16) unsigned char fsm[];
  uint4* slab = reinterpret_cast<uint4*>(fsm);
  float* bl = reinterpret_cast<float*>(slab + 2 * SLAB);  // b1 | W2[0] | W2[1]
  float* yl = bl + 3 * HID;                               // 64 floats per wave
  float* red = reinterpret_cast<float*>(slab);            // NW x NP, after the last row block
  const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  for (int i = tid; i < HID; i += NW * 64) bl[i] = a.b1[i];
  for (int i = tid; i < 2 * HID; i += NW * 64) bl[HID + i] = a.W2[i];
  const float c0 = a.b2[0], c1 = a.b2[1];
  const int64_t nblk = (a.M + NW * 32 - 1) / (NW * 32);

  auto copy_slab = [&](int ks, int buf) {
#pragma unroll
    for (int u = 0; u < (NT * 3 + NW - 1) / NW; ++u) {
      const int piece = u * NW + wid;
      if (NT * 3 % NW == 0 || piece < NT * 3)
        copy_to_lds16_s(a.frag + (size_t)ks * SLAB + piece * 64, (uint32_t)lane * 16,
                        lds_offset(slab + buf * SLAB + piece * 64));
    }
  };
  auto load_x = [&](int64_t blk, int ks, float (&v)[8]) {
    const int64_t row = (blk * NW + wid) * 32 + (lane & 31);
    const int k = ks * 16 + 8 * half;
    if (a.vec4 && row < a.M && k + 8 <= a.k2) {
      const float4* p = reinterpret_cast<const float4*>(a.x + row * a.k2 + k);
      const float4 u = p[0], w = p[1];
      v[0] = u.x, v[1] = u.y, v[2] = u.z, v[3] = u.w;
      v[4] = w.x, v[5] = w.y, v[6] = w.z, v[7] = w.w;
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = row < a.M && k + e < a.k2 ? a.x[row * a.k2 + k + e] : 0.f;
    }
  };

  float gb[NT], g0[NT], g1[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) gb[nt] = g0[nt] = g1[nt] = 0.f;
  float d0s = 0.f, d1s = 0.f, ls = 0.f;
  float xn[8];
  int buf = 0;
  copy_slab(0, 0);
  load_x(blockIdx.x, 0, xn);
  for (int64_t blk = blockIdx.x; blk < nblk; blk += gridDim.x) {
    const int64_t r0 = (blk * NW + wid) * 32;
    const float yv = r0 * 2 + lane < 2 * a.M ? a.y[r0 * 2 + lane] : 0.f;
    floatx16 acc[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[nt][i] = 0.f;
    Extent ext;
#pragma unroll 1
    for (int ks = 0; ks < a.ksteps; ++ks) {
      float xv[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) xv[e] = xn[e];
      Split8 xs;
      xs.make(xv, ext);
      __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): this step's slab has landed
      lds_barrier();
      const bool more = ks + 1 < a.ksteps;
      const int64_t nb = more ? blk : blk + gridDim.x;
      if (nb < nblk) {  // the other slab was last read in the previous step
        copy_slab(more ? ks + 1 : 0, buf ^ 1);
        load_x(nb, more ? ks + 1 : 0, xn);
      }
      const uint4* sb = slab + buf * SLAB + lane;
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        bf16x8 w[3];
#pragma unroll
        for (int s = 0; s < 3; ++s) __builtin_memcpy(&w[s], sb + (nt * 3 + s) * 64, 16);
        acc[nt] = mfma_split(xs.t, w, acc[nt]);
        if (nt & 1) __builtin_amdgcn_sched_barrier(0);  // (bounds the fragments in flight)
      }
      buf ^= 1;
    }
    if (__any(ext.beyond_terms()) || *a.bad) {  // the wave's rows again in fp32
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[nt][i] = 0.f;
      const int64_t row = r0 + (lane & 31);
#pragma unroll 1
      for (int k = half; k < a.k2; k += 2) {  // (k2 is even)
        const float xk = row < a.M ? a.x[row * a.k2 + k] : 0.f;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
          acc[nt] = __builtin_amdgcn_mfma_f32_32x32x2f32(
              xk, a.W1[(int64_t)(nt * 32 + (lane & 31)) * a.k2 + k], acc[nt], 0, 0, 0);
      }
    }
    // ---- layer 2: acc[nt][i] is unit 32 nt + (lane & 31) of row r0 + 8 (i / 4) + 4 half + i % 4
    yl[wid * 64 + lane] = yv;
    float p0[16], p1[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) p0[i] = p1[i] = 0.f;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const int u = nt * 32 + (lane & 31);
      const float b = bl[u], w0 = bl[HID + u], w1 = bl[2 * HID + u];
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const float h = fmaxf(acc[nt][i] + b, 0.f);
        acc[nt][i] = h;
        p0[i] = fmaf(h, w0, p0[i]);
        p1[i] = fmaf(h, w1, p1[i]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    // ---- the loss and its gradient at the prediction (in place of p)
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int rr = 8 * (i >> 2) + 4 * half + (i & 3);
      const bool in = r0 + rr < a.M;
      const float2 t = *reinterpret_cast<const float2*>(yl + wid * 64 + 2 * rr);
      const float e0 = half_wave_sum(p0[i]) + c0 - t.x, e1 = half_wave_sum(p1[i]) + c1 - t.y;
      p0[i] = in ? 2.f * e0 * a.inv_m : 0.f;
      p1[i] = in ? 2.f * e1 * a.inv_m : 0.f;
      d0s += p0[i];
      d1s += p1[i];
      if (in) ls = fmaf(e0, e0 * a.inv_m, fmaf(e1, e1 * a.inv_m, ls));  // the loss is a mean over rows
    }
    // ---- back to z
    float* dz = a.dZ + (r0 >> 5) * HID * 32 + lane * 4;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const int u = nt * 32 + (lane & 31);
      const float w0 = bl[HID + u], w1 = bl[2 * HID + u];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        float v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int i = q * 4 + j;
          const float h = acc[nt][i];
          v[j] = h > 0.f ? fmaf(p0[i], w0, p1[i] * w1) : 0.f;
          g0[nt] = fmaf(p0[i], h, g0[nt]);
          g1[nt] = fmaf(p1[i], h, g1[nt]);
          gb[nt] += v[j];
        }
        *reinterpret_cast<float4*>(dz + (nt * 4 + q) * 256) = make_float4(v[0], v[1], v[2], v[3]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  __syncthreads();
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {  // the two halves hold different rows
    const float b = gb[nt] + __shfl_xor(gb[nt], 32), u = g0[nt] + __shfl_xor(g0[nt], 32),
                v = g1[nt] + __shfl_xor(g1[nt], 32);
    if (half == 0) {
      red[wid * NP + nt * 32 + lane] = b;
      red[wid * NP + HID + nt * 32 + lane] = u;
      red[wid * NP + 2 * HID + nt * 32 + lane] = v;
    }
  }
  const float t0 = d0s + __shfl_xor(d0s, 32), t1 = d1s + __shfl_xor(d1s, 32),
              t2 = ls + __shfl_xor(ls, 32);
  if (lane == 0) {
    red[wid * NP + 3 * HID] = t0;
    red[wid * NP + 3 * HID + 1] = t1;
    red[wid * NP + 3 * HID + 2] = t2;
  }
  __syncthreads();
  for (int c = tid; c < NP; c += NW * 64) {
    float s = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) s += red[w * NP + c];
    a.part[(int64_t)blockIdx.x * NP + c] = s;
  }
}

// One 64 TA x 128 TB tile of dW1 = dZ^T X over the row tiles of split
// blockIdx.z.  Eight waves as 2 x 4, each 32 TA units x 32 TB features.  A
// step is 16 rows: each thread fetches its units of 8 rows x 1 column from
// global memory a step ahead, splits them once and leaves the three bf16
// terms in LDS in fragment order, double buffered, one barrier per step; each
// wave reads TA + TB fragments for TA TB tiles of products.  Row order within
// a step follows dZ's layout: lane half h, element j is row 4 h + (j & 3) +
// 8 (j >> 2).
template <int TA, int TB>
__global__ __launch_bounds__(512) void k_train_dw1(int64_t M, int k2, int hidden, int per,
                                                   const float* __restrict__ dZ,
                                                   const float* __restrict__ x,
                                                   float* __restrict__ out) {
  constexpr int TILES = 2 * TA + 4 * TB;            // 32-column tiles of A, then of B
  constexpr int U = (TILES * 64 + 511) / 512;       // 8-row units per thread
  __shared__ uint4 frag[2][TILES * 3 * 64];
  __shared__ int redo;
  const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wid >> 2, wn = wid & 3;
  const int nt_all = hidden >> 5;
  const int at0 = blockIdx.y * 2 * TA, col0 = blockIdx.x * 128 * TB;
  const int64_t tiles = (M + 31) >> 5;
  const int64_t rt0 = (int64_t)blockIdx.z * per;
  const int64_t rt1 = rt0 + per < tiles ? rt0 + per : tiles;
  const int64_t nsteps = rt1 > rt0 ? (rt1 - rt0) * 2 : 0;
  if (tid == 0) redo = 0;

  // element (row r of row tile rt, unit) of dZ
  auto dz_at = [&](int64_t rt, int tile, int r, int u) {
    return dZ[((rt * nt_all + tile) * 4 + (r >> 3)) * 256 + (((r >> 2) & 1) * 32 + u) * 4 + (r & 3)];
  };
  float v[U][8];
  auto load = [&](int64_t s) {
    const int64_t rt = rt0 + (s >> 1);
    const int q0 = (int)(s & 1) * 2;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int tile = wid + 8 * u;
      if (tile < 2 * TA) {
        const bool in = at0 + tile < nt_all;
        const float4* p = reinterpret_cast<const float4*>(dZ) +
                          ((rt * nt_all + (in ? at0 + tile : 0)) * 4 + q0) * 64 + lane;
        const float4 b = p[0], c = p[64];
        v[u][0] = b.x, v[u][1] = b.y, v[u][2] = b.z, v[u][3] = b.w;
        v[u][4] = c.x, v[u][5] = c.y, v[u][6] = c.z, v[u][7] = c.w;
      } else if (tile < TILES) {
        const int col = col0 + (tile - 2 * TA) * 32 + (lane & 31);
        const int64_t row = rt * 32 + q0 * 8 + 4 * half;
        const float* p = x + row * k2 + col;
        const bool in = col < k2;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const int dr = (j & 3) + 8 * (j >> 2);
          v[u][j] = in && row + dr < M ? p[(int64_t)dr * k2] : 0.f;
        }
      }
    }
  };
  Extent ext;
  auto stage = [&](int buf) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int tile = wid + 8 * u;
      if (tile < TILES) {
        Split8 s;
        s.make(v[u], ext);
#pragma unroll
        for (int t = 0; t < 3; ++t) __builtin_memcpy(&frag[buf][(tile * 3 + t) * 64 + lane], &s.t[t], 16);
      }
    }
  };

  floatx16 acc[TA][TB];
#pragma unroll
  for (int i = 0; i < TA; ++i)
#pragma unroll
    for (int j = 0; j < TB; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
  if (nsteps) {
    load(0);
    stage(0);
  }
  __syncthreads();
  for (int64_t s = 0; s < nsteps; ++s) {
    const bool more = s + 1 < nsteps;
    if (more) load(s + 1);
    const uint4* fb = frag[s & 1] + lane;
    bf16x8 b[TB][3];
#pragma unroll
    for (int j = 0; j < TB; ++j)
#pragma unroll
      for (int t = 0; t < 3; ++t)
        __builtin_memcpy(&b[j][t], fb + ((2 * TA + wn * TB + j) * 3 + t) * 64, 16);
#pragma unroll
    for (int i = 0; i < TA; ++i) {
      bf16x8 f[3];
#pragma unroll
      for (int t = 0; t < 3; ++t) __builtin_memcpy(&f[t], fb + ((wm * TA + i) * 3 + t) * 64, 16);
#pragma unroll
      for (int j = 0; j < TB; ++j) acc[i][j] = mfma_split(f, b[j], acc[i][j]);
    }
    if (more) stage((int)((s + 1) & 1));
    lds_barrier();
  }
  if (ext.beyond_terms()) redo = 1;
  __syncthreads();
  if (redo) {  // the tile again in fp32
    for (int i = 0; i < TA; ++i)
      for (int j = 0; j < TB; ++j)
        for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
    for (int64_t rt = rt0; rt < rt1; ++rt)
      for (int r = half; r < 32; r += 2) {
        const int64_t row = rt * 32 + r;
        float av[TA], bv[TB];
#pragma unroll
        for (int i = 0; i < TA; ++i) {
          const int t = at0 + wm * TA + i;
          av[i] = t < nt_all ? dz_at(rt, t, r, lane & 31) : 0.f;
        }
#pragma unroll
        for (int j = 0; j < TB; ++j) {
          const int col = col0 + (wn * TB + j) * 32 + (lane & 31);
          bv[j] = col < k2 && row < M ? x[row * k2 + col] : 0.f;
        }
#pragma unroll
        for (int i = 0; i < TA; ++i)
#pragma unroll
          for (int j = 0; j < TB; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[i], bv[j], acc[i][j], 0, 0, 0);
      }
  }
  out += (int64_t)blockIdx.z * hidden * k2;
#pragma unroll
  for (int i = 0; i < TA; ++i) {
    const int t = at0 + wm * TA + i;
    if (t >= nt_all) continue;
#pragma unroll
    for (int j = 0; j < TB; ++j) {
      const int col = col0 + (wn * TB + j) * 32 + (lane & 31);
      if (col >= k2) continue;
#pragma unroll
      for (int e = 0; e < 16; ++e)
        out[(int64_t)(t * 32 + 8 * (e >> 2) + 4 * half + (e & 3)) * k2 + col] = acc[i][j][e];
    }
  }
}

struct EndArgs {
  int64_t nw1;              // W1's parameters
  int64_t np;               // all parameters; entry np of theirs is the loss
  int w1_parts, head_parts;
  int k2, hidden;
  const float* w1_part;     // [w1_parts][nw1]
  const float* head_part;   // [head_parts][np + 1 - nw1]
  float* theta;
  float* m1;
  float* m2;
  uint16_t* frag;
  int* bad;
  float* loss;              // or NULL
  int adam;
  float lr, beta1, beta2, eps, c1, c2;
};

// Sums the partial gradients and updates: 64 parameters per block, four
// groups of threads over the partial sums (every fourth each), then their
// sums in order.  Gradient descent (adam = 0) or Adam with bias-corrected
// moments (c1 = 1 / (1 - beta1^t), c2 = 1 / (1 - beta2^t)).  New W1 entries
// go to the fragments too.
__global__ __launch_bounds__(256) void k_train_end(EndArgs a) {
  __shared__ float sum[4][64];
  const int64_t c = (int64_t)blockIdx.x * 64 + (threadIdx.x & 63);
  const int g = threadIdx.x >> 6;
  const bool w1 = c < a.nw1;
  if (c <= a.np) {
    const int64_t ncols = w1 ? a.nw1 : a.np + 1 - a.nw1;
    const float* p = w1 ? a.w1_part + c : a.head_part + (c - a.nw1);
    const int nb = w1 ? a.w1_parts : a.head_parts;
    float s = 0.f;
#pragma unroll 8
    for (int b = g; b < nb; b += 4) s += p[b * ncols];
    sum[g][threadIdx.x & 63] = s;
  }
  __syncthreads();
  if (g || c > a.np) return;
  const int t = threadIdx.x & 63;
  const float gi = (sum[0][t] + sum[1][t]) + (sum[2][t] + sum[3][t]);
  if (c == a.np) {
    if (a.loss) *a.loss = gi;
    return;
  }
  float w = a.theta[c];
  if (!a.adam) {
    w -= a.lr * gi;
  } else {
    const float mi = fmaf(a.beta1, a.m1[c], (1.f - a.beta1) * gi);
    const float vi = fmaf(a.beta2, a.m2[c], (1.f - a.beta2) * gi * gi);
    a.m1[c] = mi;
    a.m2[c] = vi;
    w -= a.lr * (mi * a.c1) / (sqrtf(vi * a.c2) + a.eps);
  }
  a.theta[c] = w;
  if (w1) put_w1_frag(a.frag, a.hidden >> 5, (int)(c / a.k2), (int)(c % a.k2), w, a.bad);
}

static int64_t nblocks(int64_t n, int64_t per) { return (n + per - 1) / per; }

int launch_train_init(const TrainState& s, void* stream) {
  const int k2pad = (s.k2 + 15) / 16 * 16;
  hipLaunchKernelGGL(k_w1_frag, dim3((unsigned)nblocks((int64_t)s.hidden * k2pad, 256)), dim3(256),
                     0, (hipStream_t)stream, s.theta, s.k2, s.hidden, k2pad, s.frag, s.bad);
  return hipGetLastError() == hipSuccess ? VECKM_OK : VECKM_E_HIP;
}

template <int NT, int NW>
static int launch_fwd(const TrainState& s, const FwdArgs& a, int blocks, hipStream_t st) {
  constexpr int HID = NT * 32;
  // (the block's partial sums overlay the slabs)
  const size_t lds = std::max((size_t)2 * NT * 3 * 1024, (size_t)NW * (3 * HID + 3) * 4) +
                     (size_t)(3 * HID + NW * 64) * 4;
  const void* fn = reinterpret_cast<const void*>(&k_train_fwd<NT, NW>);
  if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
    return VECKM_E_HIP;
  hipLaunchKernelGGL((k_train_fwd<NT, NW>), dim3(blocks), dim3(NW * 64), lds, st, a);
  return VECKM_OK;
}

// dW1 tiles: up to 256 units x 256 features per block.
template <int TA>
static void launch_dw1(const TrainState& s, int tb, dim3 grid, int64_t m, int per, const float* x,
                       hipStream_t st) {
  if (tb == 1)
    hipLaunchKernelGGL((k_train_dw1<TA, 1>), grid, dim3(512), 0, st, m, s.k2, s.hidden, per, s.dZ, x,
                       s.w1_part);
  else
    hipLaunchKernelGGL((k_train_dw1<TA, 2>), grid, dim3(512), 0, st, m, s.k2, s.hidden, per, s.dZ, x,
                       s.w1_part);
}

int launch_train_step(const TrainState& s, const float* x, const float* y, int64_t m, int adam,
                      float lr, float c1, float c2, float* loss, void* stream) {
  hipStream_t st = (hipStream_t)stream;
  const int k2 = s.k2, hid = s.hidden;
  float* W1 = s.theta;
  float* b1 = W1 + (int64_t)hid * k2;
  float* W2 = b1 + hid;
  float* b2 = W2 + 2 * hid;
  FwdArgs f;
  f.M = m;
  f.k2 = k2;
  f.ksteps = (k2 + 15) / 16;
  f.vec4 = k2 % 4 == 0 && reinterpret_cast<uintptr_t>(x) % 16 == 0;
  f.x = x;
  f.y = y;
  f.frag = reinterpret_cast<const uint4*>(s.frag);
  f.W1 = W1;
  f.b1 = b1;
  f.W2 = W2;
  f.b2 = b2;
  f.bad = s.bad;
  f.inv_m = 1.f / (float)m;
  f.dZ = s.dZ;
  f.part = s.head_part;
  // Rows per block: 256 (128 above 256 units, whose accumulators take more
  // than half of the register file) once they fill the chip; below that 64,
  // so that a few thousand rows still spread over many CUs.
  const int big = hid <= 256 ? 8 : 4;
  const int nw = m >= (int64_t)big * 32 * 256 ? big : 2;
  const int blocks = (int)std::min<int64_t>(s.head_blocks, nblocks(m, nw * 32));
  int rc = VECKM_E_INVAL;
  switch (hid / 64) {
#define VECKM_FWD(Q, BIG)                                                             \
  case Q:                                                                             \
    rc = nw == 2 ? launch_fwd<2 * Q, 2>(s, f, blocks, st) : launch_fwd<2 * Q, BIG>(s, f, blocks, st); \
    break;
    VECKM_FWD(1, 8) VECKM_FWD(2, 8) VECKM_FWD(3, 8) VECKM_FWD(4, 8)
    VECKM_FWD(5, 4) VECKM_FWD(6, 4) VECKM_FWD(7, 4) VECKM_FWD(8, 4)
#undef VECKM_FWD
  }
  if (rc) return rc;
  // dW1 = dZ^T X, split over rows
  const TrainTiles tt = train_tiles(hid, k2, m);
  const int64_t tiles = nblocks(m, 32);
  const int per = (int)std::max<int64_t>(2, nblocks(tiles, tt.max_splits));
  const int nsplit = (int)nblocks(tiles, per);  // (at most max_splits, the size of w1_part)
  const dim3 grid(tt.nx, tt.ny, nsplit);
  switch (tt.ta) {
    case 1: launch_dw1<1>(s, tt.tb, grid, m, per, x, st); break;
    case 2: launch_dw1<2>(s, tt.tb, grid, m, per, x, st); break;
    case 3: launch_dw1<3>(s, tt.tb, grid, m, per, x, st); break;
    default: launch_dw1<4>(s, tt.tb, grid, m, per, x, st); break;
  }
  EndArgs e;
  e.nw1 = (int64_t)hid * k2;
  e.np = e.nw1 + 3 * (int64_t)hid + 2;
  e.w1_parts = nsplit;
  e.head_parts = blocks;
  e.k2 = k2;
  e.hidden = hid;
  e.w1_part = s.w1_part;
  e.head_part = s.head_part;
  e.theta = s.theta;
  e.m1 = s.m1;
  e.m2 = s.m2;
  e.frag = s.frag;
  e.bad = s.bad;
  e.loss = loss;
  e.adam = adam;
  e.lr = lr;
  e.beta1 = 0.9f;
  e.beta2 = 0.999f;
  e.eps = 1e-8f;
  e.c1 = c1;
  e.c2 = c2;
  hipLaunchKernelGGL(k_train_end, dim3((unsigned)nblocks(e.np + 1, 64)), dim3(256), 0, st, e);
  return hipGetLastError() == hipSuccess ? VECKM_OK : VECKM_E_HIP;
}

}  // namespace veckm
