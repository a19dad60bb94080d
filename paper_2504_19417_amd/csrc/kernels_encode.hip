// Host side of the encoder: shapes, LDS needs and the dispatch over D and
// precision (the kernel is in encode_kernel.h, its instances in
// kernels_encode_*.hip).
#include "encode_kernel.h"

namespace veckm {

// Rows per chunk and LDS bytes of the encoder for a given D and wave layout
// (the host-side mirror of EncShape::CH).
static int chunk_rows(int nt, int layout) {
  const int ntw = nt < enc_max_ntw(layout) ? nt : enc_max_ntw(layout), wn = nt / ntw;
  const int wm = enc_waves(layout) / wn;
  return wm * enc_mt(layout) * 16;
}

size_t encode_lds_need(int d, int precision, int nbuf, int kp, int vol, int layout) {
  const int na = precision == VECKM_FP32 ? 4 : 2, nt = d / 16;
  return (size_t)nbuf * na * nt * 64 * 16 + (size_t)kp * 4 + (size_t)chunk_rows(nt, layout) * 4 +
         16 + (size_t)vol * 4;
}

static_assert(EncShape<4, 8, 0>::CH == 8 * kEncMt * 16 && EncShape<2, 16, 0>::CH == 4 * kEncMt * 16 &&
                  EncShape<4, 1, 0>::CH == 16 * kEncMt * 16 &&
                  EncShape<4, 8, 1>::CH == 4 * 2 * kEncMt * 16 &&
                  EncShape<4, 8, 2>::CH == 4 * 2 * kEncMt * 16 &&
                  EncShape<2, 16, 2>::CH == 2 * 2 * kEncMt * 16,
              "chunk_rows mirrors EncShape");

// (one translation unit each for the larger ones)
#define VECKM_NT(NT)                                                                              \
  extern template int launch_layout<4, NT>(const EncArgs&, const EncodeTables&, int, int, hipStream_t); \
  extern template int launch_layout<2, NT>(const EncArgs&, const EncodeTables&, int, int, hipStream_t);
VECKM_NT(1) VECKM_NT(2) VECKM_NT(3) VECKM_NT(4) VECKM_NT(8) VECKM_NT(16)
#undef VECKM_NT

template <int NA>
static int dispatch_nt(const EncArgs& a, const EncodeTables& et, int rows, int num_cus,
                       hipStream_t s) {
  switch (a.D / 16) {
    case 1: return launch_layout<NA, 1>(a, et, rows, num_cus, s);
    case 2: return launch_layout<NA, 2>(a, et, rows, num_cus, s);
    case 3: return launch_layout<NA, 3>(a, et, rows, num_cus, s);
    case 4: return launch_layout<NA, 4>(a, et, rows, num_cus, s);
    case 8: return launch_layout<NA, 8>(a, et, rows, num_cus, s);
    case 16: return launch_layout<NA, 16>(a, et, rows, num_cus, s);
    default: return VECKM_E_INVAL;
  }
}

int encode_single_rows(const EncodeTables& et) {
  if (et.bits.bx > 32) return 0;  // (a brick x row's bits are one word)
  // (in the box's space: the bit table, and a head and the bits of each row)
  const int room = box_dwords(et.brick, et.rx, et.ry, et.rt) * 4 - kLutDwords * 4;
  const int fit = room / (16 + 4 * single_row_dwords(et.KP / kKStep));
  return std::min<int>(chunk_rows(et.d / 16, et.layout), fit) & ~15;
}

int encode_rows_per_chunk(int d, int layout) { return chunk_rows(d / 16, layout); }
int encode_waves(int layout) { return enc_waves(layout); }

bool encode_fusable(const EncodeTables& et, int hidden) {
  const int nt = et.d / 16;
  if (et.layout < 2 || et.layout > 4 || (nt != 4 && nt != 8) || hidden < 64 || hidden % 32)
    return false;
  const int vol = box_dwords(et.brick, et.rx, et.ry, et.rt);
  const size_t lds = slice_table_offset(encode_lds_need(et.d, et.na == 4 ? VECKM_FP32 : VECKM_FP16,
                                                        et.nbuf, et.KP, vol, et.layout)) +
                     mlp_lds_bytes(hidden);
  return lds <= 160 * 1024;
}

int launch_encode(const Batch& bt, const Workspace& w, const EncodeTables& et, int rows,
                  int num_cus, void* stream, int32_t* rowcnt, const MlpWeights* mw) {
  EncArgs a;
  a.rowcnt = rowcnt;
  a.msteps = 0;
  a.hidden = 0;
  a.unscale = 1.f;
  a.b1 = a.W2 = a.b2 = nullptr;
  a.rowflow = nullptr;
  if (fused_rows(rows)) {
    if (!mw || !mw->W1frag || !encode_fusable(et, mw->hidden)) return VECKM_E_INVAL;
    // W1 streams in behind the table: one contiguous array
    if (mw->W1frag != et.frag + (size_t)et.KP / kKStep * et.na * (et.d / 16) * 64 * 8)
      return VECKM_E_INVAL;
    a.msteps = mw->hidden / 32;
    a.hidden = mw->hidden;
    a.unscale = et.na == 4 ? mw->unscale : 1.f;  // the bf16 W1 is not scaled
    a.b1 = mw->b1;
    a.W2 = mw->W2;
    a.b2 = mw->b2;
    a.rowflow = reinterpret_cast<float2*>(w.rowflow);
  }
  a.bt = bt;
  a.b = et.brick;
  a.bb = et.bits;
  a.rx = et.rx;
  a.ry = et.ry;
  a.rt = et.rt;
  a.K = et.K;
  a.nsteps = et.KP / kKStep;
  a.SX = box_sx(et.brick, et.rx);
  a.SY = et.brick.by + 2 * et.ry;
  a.ST = et.brick.bt + 2 * et.rt;
  a.vol = a.SX * a.SY * a.ST;
  a.D = et.d;
  a.ulist = ulist_of(w);
  a.bits = reinterpret_cast<const uint2*>(brick_bits(w));
  a.order = reinterpret_cast<const int4*>(w.order);
  a.srow = reinterpret_cast<const int2*>(w.srow);
  a.runs1 = et.runs1;
  a.lds_slices = 0;
  a.frag = reinterpret_cast<const uint4*>(et.frag);
  a.runs = et.runs;
  a.wts = et.wts;
  a.count = w.count;
  a.pairs = w.pairs;
  a.rows = w.rows;
  a.plan = w.plan;
  if (a.SX > 64) return VECKM_E_INVAL;  // 16 lanes of 4 voxels read a box row, within kGridPad
  if (et.sp > 0 && (!et.runs1 || !w.srow || et.rs > encode_single_rows(et))) return VECKM_E_INVAL;
  hipStream_t s = (hipStream_t)stream;
  return et.na == 4 ? dispatch_nt<4>(a, et, rows, num_cus, s)
                    : dispatch_nt<2>(a, et, rows, num_cus, s);
}

}  // namespace veckm
