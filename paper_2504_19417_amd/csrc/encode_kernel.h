// The encoder contraction on the gfx950 matrix cores.
//
// For a query voxel v and frequency j the window sum of Eqn. 16 (with the
// count of Eqn. 17), written over integer offsets o of the window B, is
//   S_j(v) = sum_{o in B} C[v + o] e^{i theta_j(o)},   N(v) = sum_{o in B} C[v + o],
// where C is the per-voxel event count (Eqns. 14-15 with every phase
// factored out) and theta_j(o) = A[j] . o.  The encoding is S_j(v) / N(v)
// (Algorithm 1, final step).  Pairing o with -o:
//   Re S_j = sum_{o in H} (C[v+o] + C[v-o]) cos theta_j(o)
//   Im S_j = sum_{o in H} (C[v+o] - C[v-o]) sin theta_j(o)
// with H the centre plus the lexicographically positive half of B (the
// centre's cos entry is 1/2 because it is counted as +o and -o).  Both are
// dense contractions of a [rows x |H|] matrix of small integers with a fixed
// [|H| x D] table, which is what the matrix cores do: counts are exact in
// fp16, the table is one fp16 term (VECKM_FP16) or an fp16 hi/lo pair
// (VECKM_FP32), products are exact and every sum is fp32.  N(v) is the same
// pair sums against slot weights (1 per offset, 1/2 for the centre, 0 for
// padding), summed exactly in fp32 on the vector ALU.
//
// Work decomposition: the (x, y, t) grid of every slice is cut into bricks,
// and the bricks of all slices of a call form one work list.  A persistent
// block takes the item of its number, then items from a device counter: a brick
// that holds many query voxels is taken whole (its counts plus the window halo
// read from the count grid into LDS as fp16 pairs, its query voxels in chunks of up
// to 512 rows, 256 at D = 128), the rows of all other bricks in full chunks of single rows, each with its own
// window.  The table streams through LDS, shared by the block's waves.
//
// Why single rows: a chunk costs its pass over the table whatever it holds, and
// a brick its box (70 KB at r = 5/3).  64 slices of 10k events have 5 rows per
// brick, 64 lognormal slices 33: with every brick (or items of 13 single rows
// with a count box each) the encoder took 4.96 ms (FP32 form) and 10.8 ms (FP16
// form) there, with full chunks 0.67 and 3.2 ms.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "slices.h"
#include "sync.h"
#include "veckm_internal.h"

namespace veckm {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

struct EncArgs {
  Batch bt;
  Brick b;
  Brick bb;              // of the bits (EncodeTables::bits)
  int rx, ry, rt;
  int K, nsteps;
  int SX, SY, ST, vol;
  int D;
  const uint16_t* ulist;
  const uint2* bits;  // per brick x row: low and high bits of its voxels' counts (brick_bits)
  const int4* order;  // work list of whole bricks: {brick, rows, first row, slice}
  const int2* srow;   // {slice, slice-local voxel} of each single row
  const int32_t* runs1;  // the runs' offsets, packed (make_run_triples)
  int lds_slices;     // slices whose descriptors are copied to LDS (0: read them from global)
  const uint4* frag;     // the phase table's slabs, then W1's (hidden / 32, make_w1_fragments)
  const int32_t* runs;
  const uint16_t* wts;
  const int32_t* count;
  const uint32_t* pairs;
  void* rows;
  int32_t* plan;
  int32_t* rowcnt;  // per-row neighbour counts, or NULL
  // the perceptron, when the encoder runs it (kFlow* rows)
  int msteps;           // hidden / 32
  int hidden;
  float unscale;        // 2^-shift of the hi/lo W1
  const float* b1;
  const float* W2;
  const float* b2;
  float2* rowflow;      // one flow per row
};

// Marks the rows of a work item after which its block has no other to take.
constexpr int kLastItem = 1 << 30;
// Dwords of a single row's bits: 16 per run, padded to an odd multiple of 4
// dwords so that the 16 rows of a tile read from different banks.
constexpr int kLutDwords = 512;
// Plane number of rows without a ring: no step of up to kMaxRt planes leaves
// [0, 2 kNoRing).
constexpr int kNoRing = 1 << 14;
__host__ __device__ constexpr int single_row_dwords(int nsteps) { return (nsteps | 1) * 4; }

__host__ __device__ constexpr bool fused_rows(int rows) { return rows == kFlowBF16 || rows == kFlowHiLo16; }
// LDS bytes of the perceptron's constants (b1 and both rows of W2)
__host__ __device__ constexpr size_t mlp_lds_bytes(int hidden) { return (size_t)hidden * 12; }

__device__ inline half8 as_half8(uint4 u) {
  half8 h;
  __builtin_memcpy(&h, &u, 16);
  return h;
}

// (p.lo + q.hi, p.hi + q.lo) and (p.lo - q.hi, p.hi - q.lo) on packed fp16:
// the -o run comes out of the pair layout half-swapped, and the swap is free
// (the compiler folds it into the packed add's operand selects).  Exact for
// the integer counts used here (<= 2048).
typedef _Float16 half2v __attribute__((ext_vector_type(2)));

__device__ inline uint32_t pk_sum_swapped(uint32_t p, uint32_t q) {
  half2v a, b;
  __builtin_memcpy(&a, &p, 4);
  __builtin_memcpy(&b, &q, 4);
  const half2v r = a + __builtin_shufflevector(b, b, 1, 0);
  uint32_t o;
  __builtin_memcpy(&o, &r, 4);
  return o;
}
__device__ inline uint32_t pk_diff_swapped(uint32_t p, uint32_t q) {
  half2v a, b;
  __builtin_memcpy(&a, &p, 4);
  __builtin_memcpy(&b, &q, 4);
  const half2v r = a - __builtin_shufflevector(b, b, 1, 0);
  uint32_t o;
  __builtin_memcpy(&o, &r, 4);
  return o;
}

// Round to nearest even (one instruction per pair of values).
__device__ inline uint32_t pack_bf16x2(float a, float b) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  const bf16x2 v = {(__bf16)a, (__bf16)b};
  uint32_t u;
  __builtin_memcpy(&u, &v, 4);
  return u;
}

// s_waitcnt immediate (gfx9 encoding) waiting until at most n vector memory
// operations are outstanding; expcnt and lgkmcnt are left unconstrained.
constexpr int vmcnt_imm(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4) | (15 << 8); }
// ... and until at most n (<= 15) LDS operations are outstanding (vmcnt and
// expcnt unconstrained).
constexpr int lgkmcnt_imm(int n) { return 15 | (3 << 14) | (7 << 4) | ((n & 15) << 8); }

// Waves per block and the most 16-frequency tiles one wave holds (layouts 0
// and 1; layout 2 holds up to 8).
constexpr int kEncWaves = 16;
constexpr int kEncMaxNtw = 4;
// 16-row tiles each wave holds per chunk.
constexpr int kEncMt = 2;
// With four slab buffers, take the k-steps in pairs: one barrier per pair.
constexpr bool kEncPairSteps = true;

// LDS byte offset of the slice descriptors (after `bytes` of everything else).
__host__ __device__ constexpr size_t slice_table_offset(size_t bytes) { return (bytes + 15) & ~size_t(15); }

// Wave layouts of the encoder block: 0 = 16 waves (4 per SIMD) of kEncMt
// row tiles each; 1 = 8 waves (2 per SIMD) of 2 kEncMt row tiles each
// (every table fragment read from LDS feeds twice the products; half the
// waves to hide latency); 2 = 4 waves (one per SIMD) of 2 kEncMt row tiles
// over up to 8 frequency tiles (128 frequencies: every count gather feeds
// all of a row's frequencies, every table fragment four row tiles; the
// accumulators take the register file's accumulation half); 3 = 8 waves of
// kEncMt row tiles and 4 = 16 waves of one row tile, each over every
// frequency of its rows (more waves to hide latency, 128 registers each).
constexpr int enc_waves(int L) {
  return L == 0 || L == 4 ? kEncWaves : L == 1 ? kEncWaves / 2 : L == 2 ? kEncWaves / 4 : kEncWaves / 2;
}
constexpr int enc_mt(int L) { return L == 4 ? kEncMt / 2 : L == 0 || L == 3 ? kEncMt : 2 * kEncMt; }
constexpr int enc_max_ntw(int L) { return L >= 2 ? 2 * kEncMaxNtw : kEncMaxNtw; }
// layouts whose k-steps are software-pipelined within each wave
constexpr bool enc_pipelined(int L) { return L >= 2; }

template <int NA, int NT, int L>
struct EncShape {
  static constexpr int NW = enc_waves(L);       // waves per block
  static constexpr int NTW = NT < enc_max_ntw(L) ? NT : enc_max_ntw(L);  // frequency tiles per wave
  static constexpr int WN = NT / NTW;           // waves across frequencies (layouts 0, 1: 2 at D = 128, 4 at D = 256)
  static constexpr int WM = NW / WN;            // waves across rows
  static constexpr int MT = enc_mt(L);          // 16-row tiles per wave
  static constexpr int CH = WM * MT * 16;       // rows per chunk
  static constexpr int SLAB_U4 = NA * NT * 64;  // uint4 per 32-slot slab
  static constexpr int PFW = SLAB_U4 / (NW * 64);  // copies per wave per slab
  static constexpr bool EVEN = SLAB_U4 % (NW * 64) == 0;
  static constexpr int PFU = (NA * NT / 2 + NW - 1) / NW;  // copies per wave per half slab, at most
};

// Where a slab holds array q's fragment of frequency tile nt (in fragments):
// two halves, each with half of every wave's tiles in the pipelined layouts
// (which move half slabs); see make_slot_fragments.
template <int NA, int NT>
__host__ __device__ constexpr int slab_fragment(int q, int nt) {
  if (NT < 4) return q * NT + nt;
  constexpr int HN = NT >= 8 ? 4 : 2, WN = NT / (2 * HN) > 0 ? NT / (2 * HN) : 1;
  return (((nt / HN) % 2 * NA + q) * WN + nt / (2 * HN)) * HN + nt % HN;
}

// Starts the copy of one k-step slab of the phase table from global memory
// straight into LDS (no registers; completion tracked by vmcnt).  Each wave
// moves 1 KB pieces.
template <int SLAB_U4, int NW>
__device__ inline void issue_slab(const uint4* src, uint4* dst, int wid, int lane) {
  const uint32_t voff = (uint32_t)lane * 16;
#pragma unroll
  for (int u = 0; u < (SLAB_U4 + NW * 64 - 1) / (NW * 64); ++u) {
    const int base = u * NW * 64 + wid * 64;
    if (SLAB_U4 % (NW * 64) == 0 || base < SLAB_U4)
      copy_to_lds16_s(src + base, voff, lds_offset(dst + base));
  }
}

// Waits until every slab copy of this wave except those of the newest
// `newer` slabs (0..2) has landed; vector memory loads complete in order.
template <int PFW>
__device__ inline void wait_slabs(int newer) {
  static_assert(2 * PFW <= 63, "copies in flight exceed the wait counter");
  if (newer >= 2)
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(2 * PFW));
  else if (newer == 1)
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(PFW));
  else
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
}

// The count words of one k-step for MTV row tiles: for each tile, the lane's
// two +o runs (4 consecutive voxels each, two aligned pair dwords per run)
// and their -o partners.  Only the brick's count box and the run offsets are
// read, both fixed for the brick, so the next step's words can be fetched
// while the current step multiplies.
typedef uint32_t uintx2 __attribute__((ext_vector_type(2)));
typedef uint32_t uintx4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) uint32_t lds_u32;
typedef __attribute__((address_space(3))) uintx2 lds_uint2;
typedef __attribute__((address_space(3))) uintx4 lds_uint4;

// Where a wave's single rows are in LDS; tile mt's row of this lane is mt
// strides on.  Per run of 4 voxels a row keeps 16 bits: the low bits of the
// counts (3 for 3 and more) of the 4 voxels of the +o run, their high bits,
// then the same of the -o run.
struct RowRefs {
  const lds_u32* bits;   // two runs (a lane's share of a k-step) per dword
  int stride;            // dwords from tile to tile
  const lds_uint4* head; // per row: address of its pair-grid entry (48 bits), its plane, entries
  int hstride;           // per x row and per plane
  const lds_uint2* lut;  // a run's 8 bits -> its pair dwords
  int planes;            // of the ring (more than any plane number without one)
};

typedef __attribute__((address_space(1))) uint32_t global_u32;

template <int MTV>
struct CountWords {
  uint32_t P[MTV > 0 ? MTV : 1][4], Q[MTV > 0 ? MTV : 1][4];
  __device__ inline void fetch(const int32_t* runs_l, const uint32_t* vol2, const int* rb, int ks,
                               int g) {
    fetch_at(*reinterpret_cast<const int2*>(runs_l + (ks * 4 + g) * 2), vol2, rb);
  }
  // the words of the two runs starting at box offsets ro.x and ro.y
  __device__ inline void fetch_at(int2 ro, const uint32_t* vol2, const int* rb) {
#pragma unroll
    for (int mt = 0; mt < MTV; ++mt) {
      const uint32_t* p0 = vol2 + (rb[mt] + ro.x);
      const uint32_t* p1 = vol2 + (rb[mt] + ro.y);
      const uint32_t* q0 = vol2 + (rb[mt] - ro.x - 3);
      const uint32_t* q1 = vol2 + (rb[mt] - ro.y - 3);
      P[mt][0] = p0[0];
      P[mt][1] = p0[2];
      P[mt][2] = p1[0];
      P[mt][3] = p1[2];
      Q[mt][0] = q0[2];
      Q[mt][1] = q0[0];
      Q[mt][2] = q1[2];
      Q[mt][3] = q1[0];
    }
  }
  // a quarter of a tile's words: a run (of the two at ro) of the +o or the -o side
  template <int MT_, int PIECE>
  __device__ inline void fetch_piece(int2 ro, const uint32_t* vol2, const int* rb) {
    constexpr int u = PIECE & 1;
    const int off = u ? ro.y : ro.x;
    if constexpr (PIECE < 2) {
      const uint32_t* p = vol2 + (rb[MT_] + off);
      P[MT_][2 * u] = p[0];
      P[MT_][2 * u + 1] = p[2];
    } else {
      const uint32_t* q = vol2 + (rb[MT_] - off - 3);
      Q[MT_][2 * u] = q[2];
      Q[MT_][2 * u + 1] = q[0];
    }
  }
  // pieces [I, N) of all tiles, piece k being tile k / 4's
  template <int I, int N>
  __device__ inline void fetch_pieces(int2 ro, const uint32_t* vol2, const int* rb) {
    if constexpr (I < N) {
      fetch_piece<I / 4, I % 4>(ro, vol2, rb);
      fetch_pieces<I + 1, N>(ro, vol2, rb);
    }
  }
  // the same words for single rows: from the row's bits, and from the pair
  // grid where a voxel holds 3 or more events (an entry with such a voxel lies
  // in the slice, so its row and both its halves are valid).  runs: two packed
  // runs per lane group and k-step.
  // bits_ahead requests a step's bits before gather uses them.
  uint32_t ahead[MTV > 0 ? MTV : 1];
  __device__ inline void bits_ahead(int at, const RowRefs& rr) {
#pragma unroll
    for (int mt = 0; mt < MTV; ++mt) ahead[mt] = rr.bits[mt * rr.stride + at];
  }
  __device__ inline void gather(int at, const int2* runs, const RowRefs& rr) {
#pragma unroll
    for (int mt = 0; mt < MTV; ++mt) {
      const uint32_t w = ahead[mt];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const uintx2 p = rr.lut[(w >> (16 * u)) & 255], q = rr.lut[(w >> (16 * u + 8)) & 255];
        P[mt][2 * u] = p.x;
        P[mt][2 * u + 1] = p.y;
        Q[mt][2 * u] = q.y;
        Q[mt][2 * u + 1] = q.x;
      }
      const uint32_t many = w & (w >> 4) & 0x0f0f0f0fu;
      if (__any(many != 0)) {
        const uintx4 head = rr.head[mt * rr.hstride];
        const global_u32* base =
            (const global_u32*)((uint64_t)(head.y & 0xffffu) << 32 | head.x);
        const int plane = (int)(head.y >> 16);
        const int2 ro = runs[at];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const int r = u ? ro.y : ro.x;
          const int dx = (r & 255) - 32, dy = ((r >> 8) & 255) - 32, dt = r >> 16;
          const int d = dy * (int)head.z + dx, hw = (int)head.w;
          const int p = d + (plane + dt >= rr.planes ? dt - rr.planes : dt) * hw;
          const int q = -d + (plane - dt < 0 ? rr.planes - dt : -dt) * hw;
          const uint32_t m = many >> (16 * u);
          if (m & 0x003) P[mt][2 * u] = base[p];
          if (m & 0x00c) P[mt][2 * u + 1] = base[p + 2];
          if (m & 0xc00) Q[mt][2 * u] = base[q - 1];
          if (m & 0x300) Q[mt][2 * u + 1] = base[q - 3];
        }
      }
    }
  }
};

// Pair sums and differences of one k-step's count words.
template <int MTV>
__device__ inline void pair_sums(const CountWords<MTV>& cw, half8 (&cS)[MTV > 0 ? MTV : 1],
                                 half8 (&cD)[MTV > 0 ? MTV : 1]) {
#pragma unroll
  for (int mt = 0; mt < MTV; ++mt) {
    uint4 s4, d4;
    s4.x = pk_sum_swapped(cw.P[mt][0], cw.Q[mt][0]);
    s4.y = pk_sum_swapped(cw.P[mt][1], cw.Q[mt][1]);
    s4.z = pk_sum_swapped(cw.P[mt][2], cw.Q[mt][2]);
    s4.w = pk_sum_swapped(cw.P[mt][3], cw.Q[mt][3]);
    d4.x = pk_diff_swapped(cw.P[mt][0], cw.Q[mt][0]);
    d4.y = pk_diff_swapped(cw.P[mt][1], cw.Q[mt][1]);
    d4.z = pk_diff_swapped(cw.P[mt][2], cw.Q[mt][2]);
    d4.w = pk_diff_swapped(cw.P[mt][3], cw.Q[mt][3]);
    cS[mt] = as_half8(s4);
    cD[mt] = as_half8(d4);
  }
}

// One k-step of the contraction for a wave with MTV valid row tiles: the
// count pair sums of its rows (gathered from the box), the table slab `sb`
// as A operand, and the exact neighbour count on the vector ALU.
// (G: of single rows, whose count words are looked up from bits requested in the
// step before; the next step's are requested here).
template <int NA, int NT, int L, int MTV, bool G>
__device__ inline void kstep_compute(int ks, int nsteps, const uint4* sb, const int32_t* runs_l,
                                     const uint16_t* wts_l, const uint32_t* vol2,
                                     const int (&rb)[EncShape<NA, NT, L>::MT],
                                     const RowRefs& rr,
                                     CountWords<MTV>& cw,
                                     floatx4 (&accR)[EncShape<NA, NT, L>::MT][EncShape<NA, NT, L>::NTW],
                                     floatx4 (&accI)[EncShape<NA, NT, L>::MT][EncShape<NA, NT, L>::NTW],
                                     float (&cnt)[EncShape<NA, NT, L>::MT], int wn, int lane) {
  using S = EncShape<NA, NT, L>;
  constexpr int NTW = S::NTW;
  const int g = lane >> 4;
  if constexpr (MTV > 0) {
    if constexpr (!G) {
      cw.fetch(runs_l, vol2, rb, ks, g);
    } else {  // (from bits requested a step ago)
      cw.gather(ks * 4 + g, reinterpret_cast<const int2*>(runs_l), rr);
      if (ks + 1 < nsteps) cw.bits_ahead((ks + 1) * 4 + g, rr);
    }
    // pair sums and differences of counts at +o / -o: the -o run comes out
    // of the pair layout descending and half-swapped
    half8 cS[MTV], cD[MTV];
    pair_sums<MTV>(cw, cS, cD);
    const half8 bw = *reinterpret_cast<const half8*>(wts_l + ks * 32 + 8 * g);
#pragma unroll
    for (int nt = 0; nt < NTW; ++nt) {
      half8 tf[NA];
#pragma unroll
      for (int q = 0; q < NA; ++q)
        tf[q] = as_half8(sb[slab_fragment<NA, NT>(q, wn * NTW + nt) * 64 + lane]);
#pragma unroll
      for (int mt = 0; mt < MTV; ++mt) {
        if constexpr (NA == 4) {
          accR[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(tf[0], cS[mt], accR[mt][nt], 0, 0, 0);
          accI[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(tf[2], cD[mt], accI[mt][nt], 0, 0, 0);
          accR[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(tf[1], cS[mt], accR[mt][nt], 0, 0, 0);
          accI[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(tf[3], cD[mt], accI[mt][nt], 0, 0, 0);
        } else {
          accR[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(tf[0], cS[mt], accR[mt][nt], 0, 0, 0);
          accI[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(tf[1], cD[mt], accI[mt][nt], 0, 0, 0);
        }
      }
    }
    // neighbour count: the slot weights (1, 1/2 for the centre, 0 for
    // padding) against the pair sums, exact in fp32; the lane covers its 8
    // slots of the row, the 4 lanes of a row are added after the loop
#pragma unroll
    for (int mt = 0; mt < MTV; ++mt)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        cnt[mt] = __builtin_amdgcn_fdot2(half2v{bw[2 * e], bw[2 * e + 1]},
                                         half2v{cS[mt][2 * e], cS[mt][2 * e + 1]}, cnt[mt], false);
  }
}

// The k-steps of one chunk for a wave that holds MTV valid 16-row tiles
// (0 <= MTV <= MT; no per-tile branches inside).  Every wave runs it: a wave
// without rows still moves its share of each slab and meets every barrier.
// On entry the first slab is in LDS and the next NBUF - 2 are in flight.
//
// The table is the MFMA A operand and the counts the B operand, so that the
// accumulator of a lane holds 4 consecutive frequencies of one row (the
// lane's row is lane & 15): the count of that row arrives in the same lane
// and the row is written with 16-byte stores.
template <int NA, int NT, int L, int NBUF, int MTV, bool G>
__device__ inline void chunk_ksteps(int nsteps, const uint4* frag, uint4* slab,
                                    const int32_t* runs_l, const uint16_t* wts_l,
                                    const uint32_t* vol2, const int (&rb)[EncShape<NA, NT, L>::MT],
                                    const RowRefs& rr,
                                    floatx4 (&accR)[EncShape<NA, NT, L>::MT][EncShape<NA, NT, L>::NTW],
                                    floatx4 (&accI)[EncShape<NA, NT, L>::MT][EncShape<NA, NT, L>::NTW],
                                    float (&cnt)[EncShape<NA, NT, L>::MT], int wn, int wid,
                                    int lane) {
  using S = EncShape<NA, NT, L>;
  constexpr int NW = S::NW, SLAB_U4 = S::SLAB_U4, PFW = S::PFW;
  CountWords<MTV> cw;
  if constexpr (G && MTV > 0) {
    cw.bits_ahead(lane >> 4, rr);
  }
  if constexpr (kEncPairSteps && NBUF == 4) {
    // two k-steps per barrier: the slabs of the next pair go into the two
    // buffers the previous pair used (free since the last barrier) and land
    // while this pair multiplies; on entry slabs 0 and 1 are in LDS
    for (int ks = 0; ks < nsteps; ks += 2) {
#pragma unroll
      for (int u = 2; u < 4; ++u)
        if (ks + u < nsteps)
          issue_slab<SLAB_U4, NW>(frag + (size_t)(ks + u) * SLAB_U4,
                                  slab + ((ks + u) % 4) * SLAB_U4, wid, lane);
      kstep_compute<NA, NT, L, MTV, G>(ks, nsteps, slab + (ks % 4) * SLAB_U4, runs_l, wts_l,
                                    vol2, rb, rr, cw, accR, accI, cnt, wn, lane);
      if (ks + 1 < nsteps)
        kstep_compute<NA, NT, L, MTV, G>(ks + 1, nsteps, slab + ((ks + 1) % 4) * SLAB_U4, runs_l, wts_l,
                                    vol2, rb, rr, cw, accR, accI, cnt, wn, lane);
      __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));  // the next pair has landed
      lds_barrier();
    }
  } else {
    constexpr int AHEAD = NBUF - 1;
    for (int ks = 0; ks < nsteps; ++ks) {
      // start the slab AHEAD steps out now, so that it lands during this
      // step: its buffer was last read in step ks - 1, before the last barrier
      if (ks + AHEAD < nsteps)
        issue_slab<SLAB_U4, NW>(frag + (size_t)(ks + AHEAD) * SLAB_U4,
                                slab + ((ks + AHEAD) % NBUF) * SLAB_U4, wid, lane);
      kstep_compute<NA, NT, L, MTV, G>(ks, nsteps, slab + (ks % NBUF) * SLAB_U4, runs_l, wts_l,
                                    vol2, rb, rr, cw, accR, accI, cnt, wn, lane);
      // make sure the slab of step ks + 1 has landed (slabs ks + 2 .. ks +
      // AHEAD may stay in flight)
      const int last = ks + AHEAD < nsteps - 1 ? ks + AHEAD : nsteps - 1;  // newest slab issued
      wait_slabs<PFW>(last - ks - 1 > 0 ? last - ks - 1 : 0);
      lds_barrier();
    }
  }
}

// Dispatches on the wave's number of valid row tiles (wave-uniform).
template <int NA, int NT, int L, int NBUF, int M, bool G>
__device__ inline void chunk_ksteps_n(int mtv, int nsteps, const uint4* frag, uint4* slab,
                                      const int32_t* runs_l, const uint16_t* wts_l,
                                      const uint32_t* vol2, const int (&rb)[EncShape<NA, NT, L>::MT],
                                      const RowRefs& rr,
                                      floatx4 (&accR)[EncShape<NA, NT, L>::MT][EncShape<NA, NT, L>::NTW],
                                      floatx4 (&accI)[EncShape<NA, NT, L>::MT][EncShape<NA, NT, L>::NTW],
                                      float (&cnt)[EncShape<NA, NT, L>::MT], int wn, int wid,
                                      int lane) {
  if constexpr (M == 0) {
    chunk_ksteps<NA, NT, L, NBUF, 0, G>(nsteps, frag, slab, runs_l, wts_l, vol2, rb, rr, accR, accI, cnt,
                                  wn, wid, lane);
  } else {
    if (mtv == M)
      chunk_ksteps<NA, NT, L, NBUF, M, G>(nsteps, frag, slab, runs_l, wts_l, vol2, rb, rr, accR, accI, cnt,
                                    wn, wid, lane);
    else
      chunk_ksteps_n<NA, NT, L, NBUF, M - 1, G>(mtv, nsteps, frag, slab, runs_l, wts_l, vol2, rb, rr, accR,
                                          accI, cnt, wn, wid, lane);
  }
}

// ---- layouts 2 to 4: software-pipelined k-steps ---------------------------
//
// The slabs stream through LDS in half-slab units (half of each wave's
// frequency tiles of a k-step, then one hidden tile of W1 each), four of them
// in a ring.  While unit u is in use, u + 1 has landed, u + 2 is landing and
// u + 3 is requested into the buffer u - 1 left: one barrier per unit, at
// which each wave's copies of u + 2 have landed.  Since the next unit can be
// read before the barrier, table fragments are requested TA frequency tiles
// ahead of their products across units and k-steps, and no barrier drains the
// LDS pipe.  The next step's count words are requested a few at a time behind
// the fragments of the second half's frequency tiles (LDS reads complete in order, so
// in one go they would hold up every fragment behind them).  The unit
// sequence is cyclic (table, W1, table, ...), as every chunk reads the same:
// the copies run on across chunks and work items.
//
// What bounds it: a wave reads every fragment of the slab for its 16 MT rows,
// so the block's LDS reads are NW x 32 KB (FP32 form, D = 128) per k-step at
// 128 B per cycle.  With 16 waves of one tile (layout 4) that is 4096 cycles
// against 2048 of matrix products; with 8 waves of two tiles (layout 3) it is
// 2048 against 2048.  What then remains beside the products is vector work that
// both waves of a SIMD do at the same time (pair sums, the division by the
// count), so that is spread between products where it can be (layer 2 runs
// behind the next tile's products).  1M-event slice, encoder and perceptron, when
// it replaced one slab ahead in the 16-wave layout: FP32 form 0.56 to 0.52 ms,
// FP16 form 0.37 to 0.29 ms (0.48 and 0.28 ms in passes of one case now).  Each accumulator receives exactly the products of
// layouts 0 and 1 in the same order: results are bit-identical.

// The unit stream of a block's wave (all wave-uniform): units lie back to back
// in global memory, each copied as 1 KB pieces dealt over the waves.
struct UnitRing {
  const unsigned char* src;  // this wave's first piece of unit 0
  uint32_t dst;              // LDS byte offset of that piece in buffer 0
  int units;                 // in the cycle
  int next;                  // unit to request next
  int put, get;              // ring positions of that unit and of the unit in use
};

template <int NA, int NT, int L>
__device__ inline void issue_unit(UnitRing& r, int wid, int lane) {
  using S = EncShape<NA, NT, L>;
  constexpr int PIECES = NA * NT / 2;
  const unsigned char* src = r.src + (size_t)(uint32_t)r.next * (PIECES * 1024);
  const uint32_t dst = r.dst + r.put * (PIECES * 1024);
#pragma unroll
  for (int u = 0; u < S::PFU; ++u)
    if (PIECES % S::NW == 0 || wid < PIECES)
      copy_to_lds16_s(src, (uint32_t)(lane * 16 + u * S::NW * 1024), dst + u * S::NW * 1024);
  r.put = (r.put + 1) & 3;
  r.next = r.next + 1 == r.units ? 0 : r.next + 1;
}

// What the fused perceptron needs inside a chunk (kFlow* rows).
struct FuseArgs {
  int msteps;           // W1 slabs: two hidden tiles of 16 units each
  float unscale;
  const float* mlp_l;   // LDS: b1[hidden], W2[0][hidden], W2[1][hidden]
  int hidden;
  float b20, b21;
  float2* out;          // rowflow
  int row_first;        // row index of the chunk's first row
  int nr;               // rows in the chunk
  int wm;               // this wave's row group
};

typedef __bf16 bf16x8_e __attribute__((ext_vector_type(8)));

template <int I, int N, class F>
__device__ inline void phases(F& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    phases<I + 1, N>(f);
  }
}

// The k-steps of one chunk, then (FUSE) the perceptron on its rows.  On entry
// the ring's unit in use is unit 0, which has landed for the whole block like
// unit 1, and unit 2 is requested.
template <int NA, int NT, int L, int MTV, bool FUSE, bool G>
__device__ inline void chunk_ksteps_p(int nsteps, const uint4* slab, UnitRing& ring,
                                      const int32_t* runs_l, const uint16_t* wts_l,
                                      const uint32_t* vol2, const int (&rb)[EncShape<NA, NT, L>::MT],
                                      const RowRefs& rr,
                                      floatx4 (&accR)[EncShape<NA, NT, L>::MT][EncShape<NA, NT, L>::NTW],
                                      floatx4 (&accI)[EncShape<NA, NT, L>::MT][EncShape<NA, NT, L>::NTW],
                                      float (&cnt)[EncShape<NA, NT, L>::MT], int wn, int wid,
                                      int lane, const FuseArgs& fz) {
  using S = EncShape<NA, NT, L>;
  constexpr int NTW = S::NTW, HN = NTW / 2, UNIT = S::SLAB_U4 / 2, WM = S::WM;
  // frequency tiles of table fragments in flight beyond the one in use (the
  // 16-wave layout's registers hold none: its other waves hide the wait)
  constexpr int TA = L == 4 ? 0 : NA == 2 && NTW == 8 ? 3 : 1;
  static_assert(TA <= HN && NTW % (TA + 1) == 0, "fragments in flight stay within the next unit");
  const int g = lane >> 4;
  const int2* runs2 = reinterpret_cast<const int2*>(runs_l);
  auto unit = [&](int ahead) { return slab + ((ring.get + ahead) & 3) * UNIT; };
  auto issue = [&]() { issue_unit<NA, NT, L>(ring, wid, lane); };
  // the end of a unit: this wave's copies of the next but one have landed
  // (those of the one after may stay in flight), then every wave's
  auto turn = [&]() {
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(S::PFU));
    asm volatile("s_barrier" ::: "memory");
    ring.get = (ring.get + 1) & 3;
  };
  CountWords<MTV> cw;
  int2 ro_next = make_int2(0, 0);
  half8 cS[MTV > 0 ? MTV : 1], cD[MTV > 0 ? MTV : 1];
  half8 tf[TA + 1][NA];
  auto frags = [&](int slot, const uint4* ub, int i) {  // tile i of the unit at ub
#pragma unroll
    for (int q = 0; q < NA; ++q) tf[slot][q] = as_half8(ub[((q * S::WN + wn) * HN + i) * 64 + lane]);
  };
  if constexpr (MTV > 0) {
    if constexpr (G) {
      cw.bits_ahead(g, rr);
      cw.gather(g, runs2, rr);
      if (nsteps > 1) cw.bits_ahead(4 + g, rr);
    } else {
      cw.fetch_at(runs2[g], vol2, rb);
      if (nsteps > 1) ro_next = runs2[4 + g];
    }
#pragma unroll
    for (int i = 0; i < TA; ++i) frags(i, unit(0), i);
    pair_sums<MTV>(cw, cS, cD);
  }
#pragma unroll 1
  for (int ks = 0; ks < nsteps; ++ks) {
    half8 bw;
    if constexpr (MTV > 0) {
      const uint4* u0 = unit(0);
      const uint4* u1 = unit(1);
      const uint4* u2 = unit(2);
      auto phase = [&](auto I) {
        constexpr int i = decltype(I)::value, a = i + TA;  // products of tile i, fragments of tile a
        if constexpr (a < HN) frags(a % (TA + 1), u0, a);
        else if constexpr (a < NTW) frags(a % (TA + 1), u1, a - HN);
        else frags(a % (TA + 1), u2, a - NTW);  // (past the last step: read, never used)
        if constexpr (i == 0) bw = *reinterpret_cast<const half8*>(wts_l + ks * 32 + 8 * g);
        if (ks + 1 < nsteps) {
          if constexpr (G) {
            if constexpr (i == 0) cw.gather((ks + 1) * 4 + g, runs2, rr);
            if constexpr (i == NTW - 1)
              if (ks + 2 < nsteps) cw.bits_ahead((ks + 2) * 4 + g, rr);
          } else if constexpr (i >= HN - 1 && i < NTW - 1) {
            constexpr int PP = 4 * MTV / HN > 0 ? 4 * MTV / HN : 1, k = (i - HN + 1) * PP;
            cw.template fetch_pieces<(k < 4 * MTV ? k : 4 * MTV),
                                     (k + PP < 4 * MTV ? k + PP : 4 * MTV)>(ro_next, vol2, rb);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
        const half8* t = tf[i % (TA + 1)];
        if constexpr (NA == 4) {
#pragma unroll
          for (int mt = 0; mt < MTV; ++mt) {
            accR[mt][i] = __builtin_amdgcn_mfma_f32_16x16x32_f16(t[0], cS[mt], accR[mt][i], 0, 0, 0);
            accI[mt][i] = __builtin_amdgcn_mfma_f32_16x16x32_f16(t[2], cD[mt], accI[mt][i], 0, 0, 0);
          }
#pragma unroll
          for (int mt = 0; mt < MTV; ++mt) {
            accR[mt][i] = __builtin_amdgcn_mfma_f32_16x16x32_f16(t[1], cS[mt], accR[mt][i], 0, 0, 0);
            accI[mt][i] = __builtin_amdgcn_mfma_f32_16x16x32_f16(t[3], cD[mt], accI[mt][i], 0, 0, 0);
          }
        } else {
#pragma unroll
          for (int mt = 0; mt < MTV; ++mt) {
            accR[mt][i] = __builtin_amdgcn_mfma_f32_16x16x32_f16(t[0], cS[mt], accR[mt][i], 0, 0, 0);
            accI[mt][i] = __builtin_amdgcn_mfma_f32_16x16x32_f16(t[1], cD[mt], accI[mt][i], 0, 0, 0);
          }
        }
        if constexpr (i == HN - 1) {
          // the neighbour count (see kstep_compute)
#pragma unroll
          for (int mt = 0; mt < MTV; ++mt)
#pragma unroll
            for (int e = 0; e < 4; ++e)
              cnt[mt] = __builtin_amdgcn_fdot2(half2v{bw[2 * e], bw[2 * e + 1]},
                                               half2v{cS[mt][2 * e], cS[mt][2 * e + 1]}, cnt[mt], false);
        }
        if constexpr (i == NTW - 1 && !G)
          if (ks + 2 < nsteps) ro_next = runs2[(ks + 2) * 4 + g];
        __builtin_amdgcn_sched_barrier(0);
      };
      // (copies are requested behind the first products of a unit)
      phases<0, 1>(phase);
      issue();
      phases<1, HN>(phase);
      turn();
      phases<HN, HN + 1>(phase);
      issue();
      phases<HN + 1, NTW>(phase);
      if (ks + 1 < nsteps) pair_sums<MTV>(cw, cS, cD);
    } else {
      issue();
      turn();
      issue();
    }
    turn();
  }
  if constexpr (FUSE) {
    // ---- the perceptron on the chunk's rows, still in registers (Sec. 2.1,
    //      Eqns. 5-6): x = [Re emb | Im emb] as the B operand of layer 1,
    //      W1 from the units that follow the table's (one hidden tile of 16
    //      units each), ReLU and layer 2 on the vector ALU.  The lane holds
    //      features 16 nt + 4 g + (0..3) of row lane & 15; layer-1 step kk
    //      takes frequency tiles 2kk' and 2kk' + 1 (real parts for kk < NT / 2,
    //      imaginary parts above), the order the W1 fragments were laid out in.
    //      W1 fragments are requested LA steps ahead, across units too.
    static_assert(S::WN == 1, "the fused perceptron needs every frequency of a row in one wave");
    constexpr int TERMS = NA / 2;
    constexpr int KK = NT;  // 32-feature steps of layer 1
    uint4 xh[MTV > 0 ? MTV : 1][KK], xl[TERMS == 2 && MTV > 0 ? MTV : 1][TERMS == 2 ? KK : 1];
    float p0[MTV > 0 ? MTV : 1], p1[MTV > 0 ? MTV : 1];
    if constexpr (MTV > 0) {
#pragma unroll
      for (int mt = 0; mt < MTV; ++mt) {
        float n = cnt[mt];
        n += __shfl_xor(n, 16);
        n += __shfl_xor(n, 32);
        // x / n as the encoder's rows are (exact for x = n; 0 without neighbours:
        // every sum is 0 then)
        const float rc = n > 0.f ? __builtin_amdgcn_rcpf(n) : 0.f;
        auto div = [n, rc](float x) {
          const float qq = x * rc;
          return fmaf(fmaf(-qq, n, x), rc, qq);
        };
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
          const int t0 = 2 * (kk % (NT / 2));
          const floatx4 a0 = kk < NT / 2 ? accR[mt][t0] : accI[mt][t0];
          const floatx4 a1 = kk < NT / 2 ? accR[mt][t0 + 1] : accI[mt][t0 + 1];
          float v[8] = {div(a0[0]), div(a0[1]), div(a0[2]), div(a0[3]),
                        div(a1[0]), div(a1[1]), div(a1[2]), div(a1[3])};
          if constexpr (TERMS == 2) {
            half8 h, l;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              // (the fp32 value itself is split: fused into the conversions, hi
              // and the hi that lo is taken from can round differently)
              asm("" : "+v"(v[e]));
              h[e] = (_Float16)v[e];
              l[e] = (_Float16)(v[e] - (float)h[e]);
            }
            __builtin_memcpy(&xh[mt][kk], &h, 16);
            __builtin_memcpy(&xl[mt][kk], &l, 16);
          } else {
            xh[mt][kk] = make_uint4(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]),
                                    pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7]));
          }
        }
        p0[mt] = 0.f;
        p1[mt] = 0.f;
      }
    }
    constexpr int LA = 3;
    static_assert(KK % (LA + 1) == 0 && LA <= KK, "fragments in flight stay within the next unit");
    half8 wf[LA + 1][TERMS];
    auto wfrags = [&](int slot, const uint4* ub, int kk) {
#pragma unroll
      for (int t = 0; t < TERMS; ++t) wf[slot][t] = as_half8(ub[(t * KK + kk) * 64 + lane]);
    };
    if constexpr (MTV > 0) {
#pragma unroll
      for (int i = 0; i < LA; ++i) wfrags(i, unit(0), i);
    }
    // Layer 2 of a unit runs between the products of the next: its hidden
    // values (of tile m: units 16 m + 4 g + i in this lane), b1 and W2.
    floatx4 h[MTV > 0 ? MTV : 1], hp[MTV > 0 ? MTV : 1];
    floatx4 bp, w0p, w1p;
    auto layer2 = [&](int k) {  // value k of MTV * 4
      const int mt = k >> 2, i = k & 3;
      const float hv = fmaxf(fmaf(hp[mt][i], fz.unscale, bp[i]), 0.f);
      p0[mt] = fmaf(w0p[i], hv, p0[mt]);
      p1[mt] = fmaf(w1p[i], hv, p1[mt]);
    };
    auto tile = [&](auto First) {
      constexpr bool first = decltype(First)::value;
      if constexpr (MTV > 0) {
        const uint4* u0 = unit(0);
        const uint4* u1 = unit(1);
#pragma unroll
        for (int mt = 0; mt < MTV; ++mt) h[mt] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
          if (kk + LA < KK) wfrags((kk + LA) % (LA + 1), u0, kk + LA);
          else wfrags((kk + LA) % (LA + 1), u1, kk + LA - KK);
          __builtin_amdgcn_sched_barrier(0);
          const half8* w = wf[kk % (LA + 1)];
          if constexpr (TERMS == 2) {
#pragma unroll
            for (int mt = 0; mt < MTV; ++mt)
              h[mt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w[0], as_half8(xh[mt][kk]), h[mt], 0, 0, 0);
#pragma unroll
            for (int mt = 0; mt < MTV; ++mt)
              h[mt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w[1], as_half8(xh[mt][kk]), h[mt], 0, 0, 0);
#pragma unroll
            for (int mt = 0; mt < MTV; ++mt)
              h[mt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w[0], as_half8(xl[mt][kk]), h[mt], 0, 0, 0);
          } else {
            bf16x8_e wb;
            __builtin_memcpy(&wb, &w[0], 16);
#pragma unroll
            for (int mt = 0; mt < MTV; ++mt) {
              bf16x8_e xb;
              __builtin_memcpy(&xb, &xh[mt][kk], 16);
              h[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wb, xb, h[mt], 0, 0, 0);
            }
          }
          if constexpr (!first) {
            // (the last unit's layer 2 is spread over all but the last steps)
            constexpr int PER = (4 * MTV + KK - 2) / (KK - 1);
#pragma unroll
            for (int k = kk * PER; k < (kk + 1) * PER; ++k)
              if (k < 4 * MTV) layer2(k);
          }
          if (kk == 1) issue();
          __builtin_amdgcn_sched_barrier(0);
        }
      } else {
        issue();
      }
    };
    auto keep = [&](int m) {  // tile m's sums and constants for its layer 2
      if constexpr (MTV > 0) {
        const int u = m * 16 + 4 * g;
        bp = *reinterpret_cast<const floatx4*>(fz.mlp_l + u);
        w0p = *reinterpret_cast<const floatx4*>(fz.mlp_l + fz.hidden + u);
        w1p = *reinterpret_cast<const floatx4*>(fz.mlp_l + 2 * fz.hidden + u);
#pragma unroll
        for (int mt = 0; mt < MTV; ++mt) hp[mt] = h[mt];
      }
      turn();
    };
    tile(std::true_type{});
    keep(0);
#pragma unroll 1
    for (int m = 1; m < 2 * fz.msteps; ++m) {
      tile(std::false_type{});
      keep(m);
    }
    if constexpr (MTV > 0) {
#pragma unroll
      for (int k = 0; k < 4 * MTV; ++k) layer2(k);
    }
    // ---- one flow per row: the 4 lanes of a row hold partial sums
    if constexpr (MTV > 0) {
#pragma unroll
      for (int mt = 0; mt < MTV; ++mt) {
        float f0 = p0[mt], f1 = p1[mt];
        f0 += __shfl_xor(f0, 16);
        f1 += __shfl_xor(f1, 16);
        f0 += __shfl_xor(f0, 32);
        f1 += __shfl_xor(f1, 32);
        const int r = (mt * WM + fz.wm) * 16 + (lane & 15);
        if (lane < 16 && r < fz.nr) fz.out[fz.row_first + r] = make_float2(f0 + fz.b20, f1 + fz.b21);
      }
    }
  }
}

template <int NA, int NT, int L, int M, bool FUSE, bool G>
__device__ inline void chunk_ksteps_pn(int mtv, int nsteps, const uint4* slab, UnitRing& ring,
                                       const int32_t* runs_l, const uint16_t* wts_l,
                                       const uint32_t* vol2, const int (&rb)[EncShape<NA, NT, L>::MT],
                                       const RowRefs& rr,
                                       floatx4 (&accR)[EncShape<NA, NT, L>::MT][EncShape<NA, NT, L>::NTW],
                                       floatx4 (&accI)[EncShape<NA, NT, L>::MT][EncShape<NA, NT, L>::NTW],
                                       float (&cnt)[EncShape<NA, NT, L>::MT], int wn, int wid,
                                       int lane, const FuseArgs& fz) {
  if constexpr (M == 0) {
    chunk_ksteps_p<NA, NT, L, 0, FUSE, G>(nsteps, slab, ring, runs_l, wts_l, vol2, rb, rr, accR, accI,
                                             cnt, wn, wid, lane, fz);
  } else {
    if (mtv == M)
      chunk_ksteps_p<NA, NT, L, M, FUSE, G>(nsteps, slab, ring, runs_l, wts_l, vol2, rb, rr, accR,
                                               accI, cnt, wn, wid, lane, fz);
    else
      chunk_ksteps_pn<NA, NT, L, M - 1, FUSE, G>(mtv, nsteps, slab, ring, runs_l, wts_l, vol2, rb, rr,
                                                    accR, accI, cnt, wn, wid, lane, fz);
  }
}

// The same slice in every lane: into scalar registers.
__device__ inline SliceDesc uniform(SliceDesc s) {
  int w[sizeof(SliceDesc) / 4];
  __builtin_memcpy(w, &s, sizeof(s));
#pragma unroll
  for (int i = 0; i < (int)(sizeof(SliceDesc) / 4); ++i) w[i] = __builtin_amdgcn_readfirstlane(w[i]);
  __builtin_memcpy(&s, w, sizeof(s));
  return s;
}

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef _Float16 half4v __attribute__((ext_vector_type(4)));

// The kernel's arguments, read again from where it is called (scalar loads from
// the argument segment): used straight from the parameter they are all loaded
// at the kernel's start and held, or spilled, across the k-steps.  Scalar spills
// at D = 32, 256 and 128 (FP16 form) 114, 133 and 151, so 26, 37 and 60; 5M-event
// slice 2.50 to 2.44 ms, 900k events at D = 256 2.22 to 2.14 ms (FP32 form).
__device__ inline __attribute__((always_inline)) const EncArgs& encode_args() {
  typedef __attribute__((address_space(4))) const EncArgs* args_ptr;
  args_ptr p = (args_ptr)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *(const EncArgs*)p;
}

template <int NA, int NT, int L, int NBUF, int ROWS>
__global__ __launch_bounds__(enc_waves(L) * 64) void k_encode(EncArgs) {
  const EncArgs& a = encode_args();
  using S = EncShape<NA, NT, L>;
  constexpr int NW = S::NW, NTW = S::NTW, WN = S::WN, WM = S::WM, MT = S::MT, CH = S::CH,
                SLAB_U4 = S::SLAB_U4, PFW = S::PFW;
  static_assert(NBUF == 2 || ((NBUF == 3 || NBUF == 4) && S::EVEN),
                "three or four slab buffers need slab copies split evenly over the waves");
  constexpr int AHEAD = NBUF - 1;  // slabs in flight beyond the one in use
  extern __shared__ __align__(16) unsigned char smem[];
  uint4* slab = reinterpret_cast<uint4*>(smem);
  int32_t* runs_l = reinterpret_cast<int32_t*>(slab + NBUF * SLAB_U4);
  int32_t* runs1_l = runs_l + a.nsteps * 8;
  uint16_t* wts_l = reinterpret_cast<uint16_t*>(runs1_l + a.nsteps * 8);
  // (a box voxel index has 16 bits: the other half of the rows' space keeps the plan)
  uint16_t* rowbase = wts_l + a.nsteps * 32;
  int4* plan_l = reinterpret_cast<int4*>(rowbase + CH);
  static_assert(CH * 2 >= 2 * sizeof(int4) && CH % 8 == 0, "the plan fits behind the rows");
  int32_t* item = reinterpret_cast<int32_t*>(rowbase + 2 * CH);
  // Count box as overlapping fp16 pairs: dword i holds the counts of box
  // voxels i and i + 1 of the same x row, so any run of 4 consecutive voxels
  // is two aligned dword reads.  Box rows are kRunPad voxels wider than the
  // halo on each side, so runs (padding slots included) stay inside a row.
  uint32_t* vol2 = reinterpret_cast<uint32_t*>(item + 4);
  // the perceptron's b1 and W2 (fused rows), then the slice descriptors of a
  // batch, when they fit
  constexpr bool FUSE = fused_rows(ROWS);
  static_assert(!FUSE || enc_pipelined(L), "the perceptron runs inside the pipelined layouts only");
  const size_t base_bytes = NBUF * SLAB_U4 * 16 + a.nsteps * 32 * 4 + CH * 4 + 16 + a.vol * 4;
  float* mlp_l = reinterpret_cast<float*>(smem + slice_table_offset(base_bytes));
  SliceDesc* stab = reinterpret_cast<SliceDesc*>(
      smem + slice_table_offset(base_bytes + (FUSE ? mlp_lds_bytes(a.hidden) : 0)));

  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wn = wid % WN, wm = wid / WN;
  const int KP = a.nsteps * 32;
  const int BV = a.b.bx * a.b.by * a.b.bt;
  const int D = a.D;
  // Work items are numbered: bricks in longest-first order, one at a time
  // (taking the next brick ahead of time upsets the balance of long jobs and
  // measured slower on sparse batches too); between those of several chunks and
  // the rest, the items of up to plan[5] single rows.  A block starts with the
  // item of its own number and takes the others from a shared counter, which no
  // block asks when there is none left for it: with the counter asked for every
  // item, the blocks of a call met at it and a small call waited 4 to 10 us for
  // its first item (a sliding window of 10k-event bins at D = 32: encoder 41.8
  // us, with numbered first items 22.7 us).  A brick's record holds all it needs; the slice
  // descriptors are in LDS.
  int4* item4 = reinterpret_cast<int4*>(item);
  // (one thread, the one that wrote plan_l)
  auto put_item = [&](int it) __attribute__((always_inline)) {
    const EncArgs& a = encode_args();
    const int4 p = plan_l[0], r = plan_l[1];
    const int rows = p.x, items = p.z, first = p.w, whole = r.x, per = r.y, nlong = r.z;
    const int ns = items - whole;
    int4 e = make_int4(-1, 0, 0, 0);
    if (it >= nlong && it < nlong + ns) {
      const int f = (it - nlong) * per;
      const int left = rows - first - f;
      e = make_int4(kSparseTag, left < per ? left : per, first + f, f);
    } else if (it < items) {
      e = a.order[it < nlong ? it : it - ns];
    }
    if (items <= (int)gridDim.x) e.y |= kLastItem;
    item4[0] = e;
  };
  // (the plan waits in LDS: held in registers across items, it costs the k-steps
  // some; read from memory for every item it is another latency before its record)
  const int4* plan4 = reinterpret_cast<const int4*>(a.plan);
  const int4 plan_p = plan4[0], plan_r = plan4[1];  // (on their way while LDS is filled)
  for (int k = tid; k < KP / 4; k += NW * 64) {
    runs_l[k] = a.runs[k];
    runs1_l[k] = a.runs1 ? a.runs1[k] : 0;  // (no single rows without it)
  }
  for (int k = tid; k < KP; k += NW * 64) wts_l[k] = a.wts[k];
  for (int k = tid; k < a.lds_slices * (int)(sizeof(SliceDesc) / 4); k += NW * 64)
    reinterpret_cast<int32_t*>(stab)[k] = reinterpret_cast<const int32_t*>(a.bt.table)[k];
  if constexpr (FUSE) {
    for (int k = tid; k < a.hidden; k += NW * 64) {
      mlp_l[k] = a.b1[k];
      mlp_l[a.hidden + k] = a.W2[k];
      mlp_l[2 * a.hidden + k] = a.W2[a.hidden + k];
    }
  }

  UnitRing ring;
  if constexpr (enc_pipelined(L)) {
    ring.src = reinterpret_cast<const unsigned char*>(a.frag) + wid * 1024;
    ring.dst = lds_offset(smem) + wid * 1024;
    ring.units = 2 * (a.nsteps + (FUSE ? a.msteps : 0));
    ring.next = ring.put = ring.get = 0;
#pragma unroll
    for (int v = 0; v < 3; ++v) issue_unit<NA, NT, L>(ring, wid, lane);
  }
  if (tid == 0) {
    plan_l[0] = plan_p;
    plan_l[1] = plan_r;
    put_item((int)blockIdx.x);
  }
  for (;;) {
    const EncArgs& a = encode_args();
    lds_barrier();
    const int4 cur = item4[0];
    const int bid = __builtin_amdgcn_readfirstlane(cur.x);
    if (bid < 0) break;
    const int nq = __builtin_amdgcn_readfirstlane(cur.y) & ~kLastItem;
    const bool last = (__builtin_amdgcn_readfirstlane(cur.y) & kLastItem) != 0;  // (uniform)
    const int row0 = __builtin_amdgcn_readfirstlane(cur.z);
    const int si = __builtin_amdgcn_readfirstlane(cur.w);
    const bool single = (bid & kSparseTag) != 0;  // (uniform)
    const int32_t* rl = single ? runs1_l : runs_l;

    // single rows use the box's space: the bit table, the rows' heads, their bits
    uint4* heads = reinterpret_cast<uint4*>(vol2 + kLutDwords);
    if (single) {
      const EncArgs& a = encode_args();
      // ---- single rows (from bricks with few rows): no count box; each row's
      //      window is collected as bits, so a chunk is full whatever bricks
      //      its rows are from, and sparse windows cost little memory traffic
      //      (read from the pair grid, 4 bytes a voxel, the rows of 64 slices
      //      of 10k events fetched 3.9 GB; from the bits, the encoder halved its
      //      time).  A wave takes 64 rows (a lane each) and every parts-th
      //      window row.
      const int nr16 = (nq + 15) & ~15, groups = (nr16 + 63) >> 6, parts = NW / groups;
      uint32_t* rbits = reinterpret_cast<uint32_t*>(heads + nr16);
      const int rstride = single_row_dwords(a.nsteps);
      {
        // fp16 of 0, 1, 2, 3 from the low and the high bit
        auto half_of = [](int lo, int hi) -> uint32_t {
          return lo & 1 ? (hi & 1 ? 0x4200u : 0x3c00u) : (hi & 1 ? 0x4000u : 0u);
        };
        for (int k = tid; k < kLutDwords; k += NW * 64) {
          const int e = (k >> 1) >> (2 * (k & 1));  // voxels 0, 1 or 2, 3 of pattern k / 2
          vol2[k] = half_of(e, e >> 4) | half_of(e >> 1, e >> 5) << 16;
        }
      }
      const int part = wid / groups, r = (wid % groups) * 64 + lane;
      if (part < parts && r < nr16) {
        const int2 e = a.srow[si + (r < nq ? r : 0)];  // (padding rows repeat the first)
        const SliceDesc sl =
            a.bt.nslices == 1 ? a.bt.s0 : a.lds_slices ? stab[e.x] : a.bt.table[e.x];
        const int x = e.y % sl.W, yt = e.y / sl.W, y = yt % sl.H, t = yt / sl.H;
        const bool ring = sl.tshift != 0;  // (bin t sits in plane t + tshift, wrapped)
        const int tp = t + sl.tshift < sl.T ? t + sl.tshift : t + sl.tshift - sl.T;
        uint32_t* rb = rbits + r * rstride;
        uint16_t* out = reinterpret_cast<uint16_t*>(rb);
        const int nl = a.bb.by * a.bb.bt, sx = __builtin_ctz(a.bb.bx), sy = __builtin_ctz(a.bb.by),
                  stt = __builtin_ctz(a.bb.bt);
        const int nbx = (sl.W + a.bb.bx - 1) >> sx, nby = (sl.H + a.bb.by - 1) >> sy;
        const int nc = (a.rx + 4) >> 2, nr = (2 * a.rx + 4) >> 2;  // runs of the centre / other rows
        const int ny = 2 * a.ry + 1, nwr = 1 + a.ry + a.rt * ny;
        if (part == 0) {
          const int w1 = sl.W + 1;
          const uint64_t at = reinterpret_cast<uint64_t>(
              a.pairs + sl.pair_off + ((int64_t)tp * sl.H + y) * w1 + (x + 1));
          heads[r] = make_uint4((uint32_t)at, (uint32_t)(at >> 32) | (uint32_t)(ring ? tp : kNoRing) << 16,
                                (uint32_t)w1, (uint32_t)(w1 * sl.H));
          for (int k = nc + (nwr - 1) * nr; k < a.nsteps * 8; ++k) out[k] = 0;  // padding runs
        }
        // The words of the window row at (y + dy, t + dt), brick column cx.  The
        // address is the row's own brick's plus 24-bit steps of bricks, columns
        // and x rows (single_rows_fit); outside the slice any word is read and masked (no branch,
        // so that loads are not serialised).
        const int tb = tp >> stt, yb = y >> sy, xb = x >> sx, plane = nbx * nby;
        const uint2* own = a.bits + (int64_t)(sl.brick_off + (tb * nby + yb) * nbx + xb) * nl;
        struct Line {
          int off;
          bool in;
        };
        auto line = [&](int dy, int dt) -> Line {
          const int yy = y + dy, tt = t + dt;
          const int pl = tt + sl.tshift < sl.T ? tt + sl.tshift : tt + sl.tshift - sl.T;
          const int step = __mul24((pl >> stt) - tb, plane) + __mul24((yy >> sy) - yb, nbx);
          return {(step << (sy + stt)) + ((pl & (a.bb.bt - 1)) << sy) + (yy & (a.bb.by - 1)),
                  (bool)(((unsigned)yy < (unsigned)sl.H) & ((unsigned)tt < (unsigned)sl.T))};
        };
        auto word = [&](Line ln, int cx) -> uint2 {
          const bool in = ln.in & ((unsigned)cx < (unsigned)nbx);
          const uint2 v = own[in ? ln.off + ((cx - xb) << (sy + stt)) : 0];
          return make_uint2(in ? v.x : 0u, in ? v.y : 0u);
        };
        auto put = [&](int first, int n, uint2 p, uint2 q) {
          for (int k = 0; k < n; ++k) {
            const int sp = 4 * k, sq = 4 * (n - 1 - k);
            out[first + k] = (uint16_t)(((p.x >> sp) & 15) | ((p.y >> sp) & 15) << 4 |
                                        ((q.x >> sq) & 15) << 8 | ((q.y >> sq) & 15) << 12);
          }
        };
        // window row w: its offsets, first run and number of runs
        auto window = [&](int w, int& dx, int& dy, int& dt, int& first, int& n) {
          if (w == 0) {
            dx = dy = dt = first = 0;
            n = nc;
            return;
          }
          dx = -a.rx;
          n = nr;
          first = nc + (w - 1) * nr;
          const int u = w - 1 - a.ry;
          dt = u < 0 ? 0 : 1 + u / ny;
          dy = u < 0 ? w : u % ny - a.ry;
        };
        if (a.bb.bx == 32) {
          // two words hold a run row of up to 28 voxels; several window rows
          // at a time, all loads first
          constexpr int kB = NW >= 16 ? 4 : 8;
          for (int w0 = part; w0 < nwr; w0 += kB * parts) {
            uint2 lo[kB][2], hi[kB][2];
#pragma unroll
            for (int u = 0; u < kB; ++u) {
              int dx, dy, dt, first, n;
              window(w0 + u * parts < nwr ? w0 + u * parts : 0, dx, dy, dt, first, n);
              const int xp = x + dx, xq = x - dx - 4 * n + 1;
              const Line lp = line(dy, dt), lq = line(-dy, -dt);
              lo[u][0] = word(lp, xp >> 5);
              hi[u][0] = word(lp, (xp >> 5) + 1);
              lo[u][1] = word(lq, xq >> 5);
              hi[u][1] = word(lq, (xq >> 5) + 1);
            }
#pragma unroll
            for (int u = 0; u < kB; ++u) {
              if (w0 + u * parts >= nwr) break;
              int dx, dy, dt, first, n;
              window(w0 + u * parts, dx, dy, dt, first, n);
              const int xp = x + dx, xq = x - dx - 4 * n + 1;
              auto cut = [](uint2 l, uint2 h, int sh) {
                return make_uint2(__builtin_amdgcn_alignbit(h.x, l.x, sh & 31),
                                  __builtin_amdgcn_alignbit(h.y, l.y, sh & 31));
              };
              put(first, n, cut(lo[u][0], hi[u][0], xp), cut(lo[u][1], hi[u][1], xq));
            }
          }
        } else {
          for (int w = part; w < nwr; w += parts) {
            int dx, dy, dt, first, n;
            window(w, dx, dy, dt, first, n);
            auto cut = [&](int x0, Line ln) {
              uint64_t o = 0, m = 0;
              const int cx = x0 >> sx, sh = x0 & (a.bb.bx - 1);
              for (int k = 0; k * a.bb.bx < sh + 4 * n; ++k) {
                const uint2 v = word(ln, cx + k);
                o |= (uint64_t)v.x << (k * a.bb.bx);
                m |= (uint64_t)v.y << (k * a.bb.bx);
              }
              return make_uint2((uint32_t)(o >> sh), (uint32_t)(m >> sh));
            };
            put(first, n, cut(x + dx, line(dy, dt)), cut(x - dx - 4 * n + 1, line(-dy, -dt)));
          }
        }
      }
    } else {
      const EncArgs& a = encode_args();
      // ---- the brick's count box, as overlapping fp16 pairs, from the counts
      const SliceDesc sl =
          uniform(a.bt.nslices == 1 ? a.bt.s0 : a.lds_slices ? stab[si] : a.bt.table[si]);
      const int lb = bid - sl.brick_off;
      const int bxi = lb % sl.nbx, byi = (lb / sl.nbx) % sl.nby, bti = lb / (sl.nbx * sl.nby);
      const int x = bxi * a.b.bx - a.rx - kRunPad + lane;
      const int y0 = byi * a.b.by - a.ry, tb = bti * a.b.bt - a.rt;
      const int nrows = a.SY * a.ST;
      // 16 lanes take a box row, 4 voxels each (the right neighbour's count is the
      // next lane's; the last column's is never read): a wave loads 4 rows at
      // once and a batch of them before any is used (12 instead of 6 spill).
      // Voxels outside the slice are masked; reads of up to kGridPad voxels
      // around the grid stay inside its allocation.  A row per wave and a voxel
      // per lane took 13.6k cycles for the 364 rows at r = 5/3, mostly issue
      // (1M-event slice, FP16 form, whole call 0.373 against 0.356 ms).
      const int l16 = lane & 15, xq = x + 3 * l16 - 16 * (lane >> 4);  // 4 l16 from the first column
      const int w4 = (a.SX + 3) >> 2;
      const bool whole = (a.SX & 3) == 0;
      const uint32_t inv = ((1u << 20) + a.SY - 1) / a.SY;  // rr / SY = rr inv >> 20 (rr < 2048)
      typedef int intx4u __attribute__((ext_vector_type(4), aligned(4)));
      const int32_t* cnt = a.count + sl.grid_off;
      constexpr int kR = 6;
      for (int r0 = wid * 4 + (lane >> 4); r0 - (lane >> 4) < nrows; r0 += NW * 4 * kR) {
        intx4u v[kR];
        uint32_t rows_in = 0;
#pragma unroll
        for (int u = 0; u < kR; ++u) {
          const int rr = r0 + u * NW * 4;
          const int st = (int)((uint32_t)rr * inv >> 20), y = y0 + rr - st * a.SY, t = tb + st;
          const bool in = (rr < nrows) & ((unsigned)y < (unsigned)sl.H) & ((unsigned)t < (unsigned)sl.T);
          const int tp = t + sl.tshift < sl.T ? t + sl.tshift : t + sl.tshift - sl.T;  // ring plane
          rows_in |= in ? 1u << u : 0u;
          v[u] = *reinterpret_cast<const intx4u*>(cnt + (in ? (tp * sl.H + y) * sl.W + xq : 0));
        }
#pragma unroll
        for (int u = 0; u < kR; ++u) {
          const int rr = r0 + u * NW * 4;
          const bool in = (rows_in >> u) & 1;
          float f[5];
#pragma unroll
          for (int k = 0; k < 4; ++k)
            f[k] = in && (unsigned)(xq + k) < (unsigned)sl.W ? (float)v[u][k] : 0.f;
          f[4] = __int_as_float(
              __builtin_amdgcn_update_dpp(0, __float_as_int(f[0]), 0x101, 0xf, 0xf, true));  // lane + 1
          uint32_t w[4];
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const auto h = __builtin_amdgcn_cvt_pkrtz(f[k], f[k + 1]);  // (exact: at most 1024)
            __builtin_memcpy(&w[k], &h, 4);
          }
          if (rr < nrows && l16 < w4) {
            uint32_t* to = vol2 + rr * a.SX + 4 * l16;
            if (whole) {
              *reinterpret_cast<uint4*>(to) = make_uint4(w[0], w[1], w[2], w[3]);
            } else {  // (rows end within a lane's four)
#pragma unroll
              for (int k = 0; k < 4; ++k)
                if (4 * l16 + k < a.SX) to[k] = w[k];
            }
          }
        }
      }
    }

    for (int c0 = 0; c0 < nq; c0 += CH) {
      const EncArgs& a = encode_args();
      const int nr = nq - c0 < CH ? nq - c0 : CH;  // rows in this chunk
      const int ntiles = (nr + 15) / 16;          // 16-row tiles holding rows
      // ---- voxel of each row (row q*16 + l of the chunk; padding reuses row 0)
      for (int r = tid; r < CH && !single; r += NW * 64) {
        const int rr = c0 + (r < nr ? r : 0);
        const int li = a.ulist[(int64_t)bid * BV + rr];
        const int sx = __builtin_ctz(a.b.bx), sy = __builtin_ctz(a.b.by);  // (powers of two)
        const int lx = li & (a.b.bx - 1), ly = (li >> sx) & (a.b.by - 1), lt = li >> (sx + sy);
        rowbase[r] = (uint16_t)(((lt + a.rt) * a.SY + (ly + a.ry)) * a.SX + (lx + a.rx + kRunPad));
      }
      // first slabs of the table (the pipelined layouts' are on their way)
      if constexpr (enc_pipelined(L)) {
        // units 0 and 1 (of a brick's later chunks: with the last units of the
        // chunk before) and the box have landed
        if (c0 == 0) __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
      } else if constexpr (kEncPairSteps && NBUF == 4) {
        // the first pair (and the box) has landed
#pragma unroll
        for (int u = 0; u < 2; ++u)
          if (u < a.nsteps)
            issue_slab<SLAB_U4, NW>(a.frag + (size_t)u * SLAB_U4, slab + u * SLAB_U4, wid, lane);
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
      } else {
#pragma unroll
        for (int u = 0; u < AHEAD; ++u)
          if (u < a.nsteps)
            issue_slab<SLAB_U4, NW>(a.frag + (size_t)u * SLAB_U4, slab + u * SLAB_U4, wid, lane);
        wait_slabs<PFW>((a.nsteps < AHEAD ? a.nsteps : AHEAD) - 1);  // slab 0 (and the box) landed
      }
      lds_barrier();

      // tiles are dealt round-robin over the row waves, so a short chunk
      // spreads evenly and fully padded tiles are skipped
      int mtv = 0;
      int rb[MT];  // voxel index of each row in the volume
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        const int q = mt * WM + wm;
        if (q < ntiles) mtv = mt + 1;
        rb[mt] = single ? 0 : rowbase[q * 16 + (lane & 15)];
      }
      mtv = __builtin_amdgcn_readfirstlane(mtv);
      RowRefs rr;
      if (single) {
        const int r = wm * 16 + (lane & 15);
        const int rstride = single_row_dwords(a.nsteps);
        rr.planes = a.bt.nslices == 1 && a.bt.s0.tshift != 0 ? a.bt.s0.T : 2 * kNoRing;
        rr.lut = (const lds_uint2*)vol2;
        rr.head = (const lds_uint4*)(heads + r);
        rr.hstride = WM * 16;
        rr.bits = (const lds_u32*)(heads + ((nq + 15) & ~15)) + r * rstride;
        rr.stride = WM * 16 * rstride;
      }

      floatx4 accR[MT][NTW], accI[MT][NTW];
      float cnt[MT];
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        cnt[mt] = 0.f;
#pragma unroll
        for (int nt = 0; nt < NTW; ++nt) {
          accR[mt][nt] = floatx4{0.f, 0.f, 0.f, 0.f};
          accI[mt][nt] = floatx4{0.f, 0.f, 0.f, 0.f};
        }
      }
      if constexpr (enc_pipelined(L)) {
        FuseArgs fz;
        fz.msteps = FUSE ? a.msteps : 0;
        fz.unscale = a.unscale;
        fz.mlp_l = mlp_l;
        fz.hidden = a.hidden;
        fz.b20 = FUSE ? a.b2[0] : 0.f;
        fz.b21 = FUSE ? a.b2[1] : 0.f;
        fz.out = a.rowflow;
        fz.row_first = row0 + c0;
        fz.nr = nr;
        fz.wm = wm;
        if (single)
          chunk_ksteps_pn<NA, NT, L, MT, FUSE, true>(mtv, a.nsteps, slab, ring, rl, wts_l,
                                                           vol2, rb, rr, accR, accI, cnt, wn, wid,
                                                           lane, fz);
        else
          chunk_ksteps_pn<NA, NT, L, MT, FUSE, false>(mtv, a.nsteps, slab, ring, rl, wts_l,
                                                            vol2, rb, rr, accR, accI, cnt, wn, wid,
                                                            lane, fz);
        if constexpr (FUSE) continue;  // flows written; no rows leave the chip
      } else if (single) {
        chunk_ksteps_n<NA, NT, L, NBUF, MT, true>(mtv, a.nsteps, a.frag, slab, rl, wts_l, vol2, rb,
                                                  rr, accR, accI, cnt, wn, wid, lane);
      } else {
        chunk_ksteps_n<NA, NT, L, NBUF, MT, false>(mtv, a.nsteps, a.frag, slab, rl, wts_l, vol2,
                                                   rb, rr, accR, accI, cnt, wn, wid, lane);
      }

      const EncArgs& out_args = encode_args();
      // ---- normalise by the neighbour count and write the rows: the lane
      //      holds frequencies 16 nt + 4 (lane >> 4) + (0..3) of row lane & 15
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        if (mt >= mtv) continue;
        const int r = (mt * WM + wm) * 16 + (lane & 15);
        // the row's count: the partial sums of its 4 lanes (exact integers)
        float n = cnt[mt];
        n += __shfl_xor(n, 16);
        n += __shfl_xor(n, 32);
        if (r >= nr) continue;
        if (out_args.rowcnt && wn == 0 && lane < 16) out_args.rowcnt[row0 + c0 + r] = (int)n;
        const float rc = __builtin_amdgcn_rcpf(n);
        // x / n: reciprocal estimate plus one residual correction (exact for
        // x = n, so an all-ones feature still gives exactly 1).  A query of a
        // sliding window can have no event in its neighbourhood (n = 0): its
        // encoding is zero.
        auto div = [n, rc](float x) {
          const float qq = x * rc;
          return n > 0.f ? fmaf(fmaf(-qq, n, x), rc, qq) : 0.f;
        };
        const int64_t u = (int64_t)(row0 + c0 + r) * (2 * D);
#pragma unroll
        for (int nt = 0; nt < NTW; ++nt) {
          const int j = (wn * NTW + nt) * 16 + 4 * (lane >> 4);
          floatx4 re, im;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            re[i] = div(accR[mt][nt][i]);
            im[i] = div(accI[mt][nt][i]);
          }
          // plain stores: a lane writes 8 or 16 bytes of a row and the other
          // lanes and frequency tiles complete its lines, which L2 merges
          // before they reach HBM (streaming stores measured 1.4-2x the
          // row bytes in HBM writes)
          if constexpr (ROWS == kRowsBF16) {
            uint16_t* out = static_cast<uint16_t*>(out_args.rows);
            u32x2 pr, pi;
            pr.x = pack_bf16x2(re[0], re[1]);
            pr.y = pack_bf16x2(re[2], re[3]);
            pi.x = pack_bf16x2(im[0], im[1]);
            pi.y = pack_bf16x2(im[2], im[3]);
            *reinterpret_cast<u32x2*>(out + u + j) = pr;
            *reinterpret_cast<u32x2*>(out + u + D + j) = pi;
          } else if constexpr (ROWS == kRowsHiLo16) {
            // fp16 hi = rne(v), lo = rne(v - hi) (v - hi is exact in fp32):
            // 22 significant bits in the perceptron's operands.  Each group
            // of 4 consecutive row elements becomes one 16-byte unit [hi x 4,
            // lo x 4], so a row keeps the fp32 row's size and a lane writes
            // one unit for its 4 real and one for its 4 imaginary parts.
            _Float16* out = static_cast<_Float16*>(out_args.rows);
            const int64_t u2 = u * 2;
            half8 ur, ui;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              ur[i] = (_Float16)re[i];
              ur[4 + i] = (_Float16)(re[i] - (float)ur[i]);
              ui[i] = (_Float16)im[i];
              ui[4 + i] = (_Float16)(im[i] - (float)ui[i]);
            }
            *reinterpret_cast<half8*>(out + u2 + 2 * j) = ur;
            *reinterpret_cast<half8*>(out + u2 + 2 * (D + j)) = ui;
          } else {
            float* out = static_cast<float*>(out_args.rows);
            *reinterpret_cast<floatx4*>(out + u + j) = re;
            *reinterpret_cast<floatx4*>(out + u + D + j) = im;
          }
        }
      }
    }
    if (last) break;
    lds_barrier();  // (the next item's rows, box and record take this one's place)
    if (tid == 0) put_item((int)gridDim.x + atomicAdd(&a.plan[1], 1));
  }
  // (no copy into LDS outlives the block)
  __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
}

template <int NA, int NT, int L, int NBUF>
static size_t encode_lds_bytes(const EncodeTables& et, int vol) {
  using S = EncShape<NA, NT, L>;
  return (size_t)NBUF * S::SLAB_U4 * 16 + (size_t)et.KP * 2 + (size_t)et.KP * 2 +
         (size_t)S::CH * 4 + 16 + (size_t)vol * 4;
}

template <int NA, int NT, int L, int NBUF, int ROWS>
static int launch_rows(const EncArgs& a, const EncodeTables& et, int num_cus, hipStream_t s) {
  constexpr bool FUSE = fused_rows(ROWS);
  size_t lds = encode_lds_bytes<NA, NT, L, NBUF>(et, a.vol);
  if (FUSE) lds = slice_table_offset(lds) + mlp_lds_bytes(a.hidden);
  if (lds > 160 * 1024) return VECKM_E_INVAL;
  // a batch's slice descriptors go to LDS when they fit beside the rest
  EncArgs b = a;
  b.lds_slices = 0;
  const size_t with_tab = slice_table_offset(lds) + (size_t)a.bt.nslices * sizeof(SliceDesc);
  if (a.bt.nslices > 1 && with_tab <= 160 * 1024) {
    b.lds_slices = a.bt.nslices;
    lds = with_tab;
  }
  const void* fn = reinterpret_cast<const void*>(&k_encode<NA, NT, L, NBUF, ROWS>);
  if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
    return VECKM_E_HIP;
  // as many blocks as a CU holds at once, by LDS and by the kernel's registers
  // (a block that has to wait for another's end would hold back the item of its
  // number: 16 waves of more than 64 registers fit once)
  static const int by_regs = [] {
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_encode<NA, NT, L, NBUF, ROWS>,
                                                        EncShape<NA, NT, L>::NW * 64, 0) == hipSuccess)
      return n;
    (void)hipGetLastError();
    return 1;
  }();
  const int per_cu = std::min((int)((160 * 1024) / lds), by_regs);
  int grid = num_cus * (per_cu < 1 ? 1 : (per_cu > 2 ? 2 : per_cu));
  // no more blocks than items: bricks of sp rows or more and items of 16 single
  // rows or more (the last one aside), or every brick with a row
  const int sp = single_rows_below(b.bt, et, num_cus, b.bt.s0.tshift != 0);
  const int items = sp > 0 ? b.bt.m / std::min(sp, 16) + 1 : std::min(b.bt.nbricks, b.bt.m);
  if (grid > items) grid = items;
  constexpr int threads = EncShape<NA, NT, L>::NW * 64;
  hipLaunchKernelGGL((k_encode<NA, NT, L, NBUF, ROWS>), dim3(grid), dim3(threads), lds, s, b);
  return hipGetLastError() == hipSuccess ? VECKM_OK : VECKM_E_HIP;
}

template <int NA, int NT, int L, int NBUF>
static int launch_t(const EncArgs& a, const EncodeTables& et, int rows, int num_cus,
                    hipStream_t s) {
  if (rows == kRowsHiLo16 && NA != 4) return VECKM_E_INVAL;  // hi/lo rows: the FP32 form only
  constexpr int HL = NA == 4 ? kRowsHiLo16 : kRowsF32;
  if (fused_rows(rows)) {
    // the perceptron inside the encoder: one wave holds all of a row's frequencies
    if constexpr (enc_pipelined(L) && EncShape<NA, NT, L>::WN == 1) {
      constexpr int FR = NA == 4 ? kFlowHiLo16 : kFlowBF16;
      if (rows != FR) return VECKM_E_INVAL;
      return launch_rows<NA, NT, L, NBUF, FR>(a, et, num_cus, s);
    }
    return VECKM_E_INVAL;
  }
  if (rows == kRowsBF16) return launch_rows<NA, NT, L, NBUF, kRowsBF16>(a, et, num_cus, s);
  if (rows == kRowsHiLo16) return launch_rows<NA, NT, L, NBUF, HL>(a, et, num_cus, s);
  return launch_rows<NA, NT, L, NBUF, kRowsF32>(a, et, num_cus, s);
}

template <int NA, int NT, int L>
static int launch_nb(const EncArgs& a, const EncodeTables& et, int rows, int num_cus,
                     hipStream_t s) {
  if constexpr (enc_pipelined(L)) {  // a ring of four half slabs: the space of two
    if (et.nbuf != 2) return VECKM_E_INVAL;
    return launch_t<NA, NT, L, 2>(a, et, rows, num_cus, s);
  } else {
    if constexpr (EncShape<NA, NT, L>::EVEN) {
      if (et.nbuf == 4) return launch_t<NA, NT, L, 4>(a, et, rows, num_cus, s);
      if (et.nbuf == 3) return launch_t<NA, NT, L, 3>(a, et, rows, num_cus, s);
    }
    return launch_t<NA, NT, L, 2>(a, et, rows, num_cus, s);
  }
}

template <int NA, int NT>
int launch_layout(const EncArgs& a, const EncodeTables& et, int rows, int num_cus,
                         hipStream_t s) {
  // the 8- and 4-wave layouts only where a wave holds several frequency tiles
  if constexpr (NT >= 4) {
    if (et.layout == 1) return launch_nb<NA, NT, 1>(a, et, rows, num_cus, s);
    if (et.layout == 2) return launch_nb<NA, NT, 2>(a, et, rows, num_cus, s);
    if (et.layout == 3) return launch_nb<NA, NT, 3>(a, et, rows, num_cus, s);
  }
  if constexpr (NT == 4 || NT == 8)
    if (et.layout == 4) return launch_nb<NA, NT, 4>(a, et, rows, num_cus, s);
  return launch_nb<NA, NT, 0>(a, et, rows, num_cus, s);
}

}  // namespace veckm
