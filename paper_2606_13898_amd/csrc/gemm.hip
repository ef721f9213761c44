// Projections of the block (QKV, attention output, MLP up and down): C = A W^T on the ragged
// packed sequence, image rows with the image-stream weights and text rows with the text-stream
// weights, tiles never straddling a segment.  Epilogues fuse the bias, the tanh-GELU, and the
// gated residual update of the float32 stream z; for the FP8 block's QKV projection, the q and k
// columns leave as E4M3 codes with a power-of-two scale per (row, head).
//
// bf16 path (k_gemm8): one persistent workgroup of 8 waves per CU, 256 x 256 or 192 x 192 tiles (chosen
// on the device from the row counts), K through LDS in 128-byte windows filled by direct global->LDS
// loads, fragments read half a window ahead of their MFMAs.
// FP8 path (k_gemm8_fp8): the same loop on E4M3 codes, 192 x 192 tiles, or 256 x 256 for the QKV projection
// (which writes FP8 q / k with one scale per row and head: a wave's 128 columns hold whole heads).
// Both: whole data-parallel waves of tiles run first, then a stream-K remainder; cut tiles leave fp32
// partials that a fixup kernel adds in a fixed order before the epilogue.
// float32 path: v_mfma_f32_16x16x4_f32 straight from global memory, K split over a workgroup's waves.
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace hilo {

// tanh-approximated GELU, 0.5 u (1 + tanh(y)) with y = sqrt(2/pi) (u + 0.044715 u^3), evaluated
// through the identity 0.5 (1 + tanh(y)) = 1 / (1 + exp(-2y)): one hardware exp2 and one
// reciprocal (about one ulp each) instead of a full tanh.  Very negative u gives exp2 -> inf and
// the result -0; very positive u gives exp2 -> 0 and the result u.
HILO_DEV float gelu_tanh(float u) {
  constexpr float c = -2.0f * 0.7978845608028654f * 1.4426950408889634f;  // -2 sqrt(2/pi) log2(e)
  const float t = c * u * (1.0f + 0.044715f * u * u);
  return u * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(t));
}

// Row range of a row tile; tiles of a sample are [image tiles][text tiles].
struct TileRows {
  int s, sigma, row0, nrows;
};

template <int EPI, bool BF16OUT>
HILO_DEV void epilogue4(const GemmProblem &p, const TileRows &tr, int m, int n, const float *acc) {
  // m: output row, n: first of 4 consecutive columns (n + 3 < N guaranteed by N % 4 == 0)
  float b[4];
  if (BF16OUT) {
    const uint2 bu = *reinterpret_cast<const uint2 *>(
        reinterpret_cast<const uint16_t *>(p.bias[tr.sigma]) + n);
    b[0] = __uint_as_float(bu.x << 16); b[1] = __uint_as_float(bu.x & 0xffff0000u);
    b[2] = __uint_as_float(bu.y << 16); b[3] = __uint_as_float(bu.y & 0xffff0000u);
  } else {
    const float4 bf = *reinterpret_cast<const float4 *>(reinterpret_cast<const float *>(p.bias[tr.sigma]) + n);
    b[0] = bf.x; b[1] = bf.y; b[2] = bf.z; b[3] = bf.w;
  }
  float v[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = acc[e] + b[e];
  if constexpr (EPI == EPI_RESID) {
    const float4 gt = *reinterpret_cast<const float4 *>(
        p.mod + (size_t(tr.s * 2 + tr.sigma) * 6 + p.gate_idx) * p.D + n);
    float4 *zp = reinterpret_cast<float4 *>(p.z + size_t(m) * p.ldz + n);
    float4 zv = *zp;
    zv.x += gt.x * v[0];
    zv.y += gt.y * v[1];
    zv.z += gt.z * v[2];
    zv.w += gt.w * v[3];
    *zp = zv;
  } else {
    if constexpr (EPI == EPI_GELU) {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = gelu_tanh(v[e]);
    }
    if (BF16OUT) {
      uint2 u;
      u.x = pack_bf16x2(v[0], v[1]);
      u.y = pack_bf16x2(v[2], v[3]);
      *reinterpret_cast<uint2 *>(reinterpret_cast<uint16_t *>(p.out) + size_t(m) * p.ldo + n) = u;
    } else {
      *reinterpret_cast<float4 *>(reinterpret_cast<float *>(p.out) + size_t(m) * p.ldo + n) =
          make_float4(v[0], v[1], v[2], v[3]);
    }
  }
}

// ------------------------------------------------------------------------------- bf16 MFMA

// One 16-byte global load per lane straight into LDS: lane l of the wave lands at byte 16*l of
// the wave's 1 KiB destination (the destination base is uniform, held in M0).
HILO_DEV void g2lds16(const void *g, void *lds_wave_base) {
  __builtin_amdgcn_global_load_lds(g, (__attribute__((address_space(3))) void *)lds_wave_base, 16, 0, 0);
}

// Active row tiles of the ragged problem: per sample, ceil(image rows / BM) image tiles then
// ceil(L / BM) text tiles.  Only the device knows the row counts, so every workgroup walks the
// (few) segments itself.
HILO_DEV int row_tiles_total(const GemmProblem &p, int BM) {
  int R = 0;
  for (int s = 0; s < p.B; ++s) {
    const int nimg = cu_at(p.cu, s + 1) - p.L - cu_at(p.cu, s);
    R += (nimg + BM - 1) / BM + (p.L + BM - 1) / BM;
  }
  return R;
}

HILO_DEV TileRows decode_row_tile(const GemmProblem &p, int BM, int r) {
  TileRows tr{0, 0, 0, 0};
  for (int s = 0; s < p.B; ++s) {
    const int lo = cu_at(p.cu, s), hi = cu_at(p.cu, s + 1), ts = hi - p.L;
    const int ti = (ts - lo + BM - 1) / BM, tt = (p.L + BM - 1) / BM;
    if (r < ti) {
      tr = TileRows{s, 0, lo + r * BM, min(BM, ts - (lo + r * BM))};
      break;
    }
    r -= ti;
    if (r < tt) {
      tr = TileRows{s, 1, ts + r * BM, min(BM, hi - (ts + r * BM))};
      break;
    }
    r -= tt;
  }
  return tr;
}

// Schedule of the projections over P = kGemmWorkgroups persistent workgroups (one per CU; a constant, so
// that the divisions by it are shifts and the prologue of every launch stays short).  A unit is one
// K piece of one output tile: tiles are cut into s pieces when there are fewer tiles than
// workgroups (s = ceil(P / tiles), at most one K step per piece), else s = 1.  Units are ordered
// piece-major, row tile fastest within a piece.  The first floor(U / P) * P units run
// data-parallel in whole waves -- the workgroups of an XCD then work on neighbouring tiles at the
// same K step, so its L2 serves each weight and activation slice to all of them.  The
// remaining units (all of the same K length) are spread evenly over the P workgroups stream-K,
// so no CU idles through a partial last wave.  A unit not finished in one place leaves an fp32
// partial tile (data-parallel unit u: slot u; stream-K range of workgroup w: slots P + 2w for its
// first unit and P + 2w + 1 for its second); gemm_fix adds the partials of each such tile in a
// fixed order and runs the epilogue -- deterministic, and no workgroup ever waits for another.
struct SkPlan {
  int R, TN, T, nk;  // row tiles, column tiles, tiles, K steps
  int s, U, dp;    // pieces per tile, units, data-parallel units
  int len;         // K steps of a stream-K unit
  long long I;     // stream-K iterations
  int Pk;          // workgroups sharing them (0 .. Pk-1; the others get empty ranges)
};

// A problem with fewer tiles than workgroups and at most this many K steps runs one whole tile per
// workgroup (some CUs idle) instead of cutting tiles into K pieces: for short K the partial tiles
// and their fixup cost more than the idle CUs.
constexpr int kNoSplitSteps = 64;

// Stream-K ranges hold at least this many K steps: every range cut leaves a partial tile (256 KiB
// at 256 x 256) that the fixup reads back, so a short tail goes to fewer workgroups.
constexpr int kSkMinSteps = 12;

// Whether T tiles of nk K steps run whole.
HILO_DEV bool runs_whole(int T, int nk) {
  constexpr int P = kGemmWorkgroups;
  // a stream-K tail costs a partial tile (144 or 256 KiB) per piece; when the last wave holds at
  // least half of P tiles, whole tiles in ceil(T / P) waves finish sooner
  const bool whole_waves = T >= P && (T % P == 0 || 2 * (T % P) >= P);
  // a single wave that fills at least 7/8 of the workgroups also runs whole tiles (cutting K would
  // add a partial per tile to save at most an eighth)
  const bool full_wave = T < P && 8 * T >= 7 * P;
  return (T < P && nk <= kNoSplitSteps) || whole_waves || full_wave;
}

// The plan of R row tiles of the problem on BN-column tiles.
HILO_DEV SkPlan sk_plan(const GemmProblem &p, int R, int BN, int kstep = 64) {
  constexpr int P = kGemmWorkgroups;
  SkPlan q;
  q.R = R;
  q.TN = (p.N + BN - 1) / BN;
  q.T = q.R * q.TN;
  q.nk = p.K / kstep;
  if (runs_whole(q.T, q.nk)) {
    q.s = 1;
    q.U = q.dp = q.T;
    q.len = q.nk;
    q.I = 0;
    q.Pk = P;
    return q;
  }
  q.s = (q.T >= P || q.T == 0) ? 1 : min((P + q.T - 1) / q.T, q.nk);
  q.U = q.T * q.s;
  q.dp = q.U / P * P;
  // the stream-K units all lie in the last piece (or every piece is one K step long)
  const int tail = q.U - q.dp;
  const int pc = tail > 0 ? q.dp / q.T : 0;
  q.len = (pc + 1) * q.nk / q.s - pc * q.nk / q.s;
  q.I = (long long)tail * q.len;
  // at least one workgroup per tail unit, so no range is longer than a unit and a range touches at
  // most two units (the two partial slots of its workgroup)
  q.Pk = int(min((long long)P, max((long long)tail, (q.I + kSkMinSteps - 1) / kSkMinSteps)));
  return q;
}

struct SkRange {
  long long beg, end;
};

// Workgroup w's stream-K range under plan q (empty past the plan's Pk workgroups).
HILO_DEV SkRange sk_range(const SkPlan &q, int w) {
  if (w >= q.Pk || q.I == 0) return SkRange{q.I, q.I};
  return SkRange{q.I * w / q.Pk, q.I * (w + 1) / q.Pk};
}

// The workgroup whose stream-K range holds iteration a.
HILO_DEV int sk_owner(long long I, int P, long long a) { return int(((a + 1) * P - 1) / I); }

HILO_DEV int piece_k0(const SkPlan &q, int piece) { return piece * q.nk / q.s; }

// Tile t -> (row tile, column tile): groups of kTileGroupRows row tiles by all column tiles, row
// tile fastest within a group, so one XCD's 32 workgroups of a wave (consecutive ids, xcd_remap)
// cover 8 row tiles by 4 column tiles: 12 operand slices per K step, the least any 32 tiles need,
// instead of 18 in plain row-fastest order over 15 row tiles.
constexpr int kTileGroupRows = 8;

HILO_DEV void tile_coords(const SkPlan &q, int t, int &r, int &tn) {
  const int grp = t / (kTileGroupRows * q.TN), in = t - grp * (kTileGroupRows * q.TN);
  const int gm = min(kTileGroupRows, q.R - grp * kTileGroupRows);
  r = grp * kTileGroupRows + in % gm;
  tn = in / gm;
}

// Work items of one workgroup, in order: its data-parallel units (u = pid, pid + P, ...), then the
// pieces of its stream-K range.  An item is (tile, 64-deep K steps [kb, ke), partial slot or null
// for a tile finished here).
struct SkItem {
  int t, kb, ke;
  float *slot;
  bool valid;
};

struct SkCursor {
  int u;          // next data-parallel unit
  long long it;   // next stream-K iteration
};

HILO_DEV SkItem sk_next_item(SkCursor &c, const SkPlan &q, const SkRange &rg, int pid, float *part,
                             size_t part_floats) {
  constexpr int P = kGemmWorkgroups;
  SkItem x{0, 0, 0, nullptr, false};
  if (c.u < q.dp) {
    const int pc = q.s == 1 ? 0 : c.u / q.T;
    x.t = c.u - pc * q.T;
    x.kb = q.s == 1 ? 0 : piece_k0(q, pc);
    x.ke = q.s == 1 ? q.nk : piece_k0(q, pc + 1);
    x.slot = q.s == 1 ? nullptr : part + size_t(c.u) * part_floats;
    x.valid = true;
    c.u += P;
  } else if (c.it < rg.end) {
    const long long v = c.it / q.len;
    const int k0 = int(c.it - v * q.len);
    const int k1 = int(min((long long)q.len, k0 + (rg.end - c.it)));
    const int uu = q.dp + int(v);
    const int pc = uu / q.T;
    x.t = uu - pc * q.T;
    x.kb = piece_k0(q, pc) + k0;
    x.ke = piece_k0(q, pc) + k1;
    const bool whole = q.s == 1 && k0 == 0 && k1 == q.len;
    x.slot = whole ? nullptr : part + (size_t(P) + size_t(pid) * 2 + (c.it == rg.beg ? 0 : 1)) * part_floats;
    x.valid = true;
    c.it += k1 - k0;
  }
  return x;
}

// Partial tiles of a BM x BN tile on WM x WN waves, in the 16 x 16 fragment order the fixup
// reads, and the fixup's epilogue of one fragment row.
// CONTIG: a lane's columns of all fragment columns are consecutive (16 x 16 blocks), instead of 4 of every 16
// (the 32 x 32 blocks of the FP8 QKV projection).
template <int BM, int BN, int WM, int WN, bool CONTIG = false>
struct SkTile {
  static constexpr int NW = WM * WN;
  static constexpr int TM = BM / WM / 16;
  static constexpr int TN = BN / WN / 16;
  static constexpr int CS = CONTIG ? 4 : 16;       // columns between fragment columns
  static constexpr int CL = CONTIG ? 4 * TN : 4;   // columns between the lane groups
  static constexpr size_t kPartFloats = size_t(BM) * BN;

  // partial-sum slot layout: register order, one float4 per lane per (wave, i, j)
  HILO_DEV static size_t part_index(int wid, int i, int j, int lane) {
    return ((size_t(wid) * TM * TN + i * TN + j) * 64 + lane) * 4;
  }

  // The FP8 q / k codes of fragment row i0 of wave wid (the whole-tile form is epilogue32_qk8):
  // the wave's BN / WN columns hold whole heads; a row's columns of one head are spread over the 4
  // lanes l % 16 + 16 m, each holding 4 columns of every 16.
  HILO_DEV static void epilogue_row_qk8(const GemmProblem &p, const TileRows &tr, int n0, int wid, int i0,
                                        int lane, const f32x4 (&acc)[TN]) {
    const int rl = (wid / WN) * (BM / WM) + i0 * 16 + (lane & 15);
    const int wc0 = n0 + (wid % WN) * (BN / WN);
    const int cbase = wc0 + 4 * (lane >> 4);
    const int hd = p.head_dim, jph = hd / 16;  // fragment columns per head
    const uint16_t *bias = reinterpret_cast<const uint16_t *>(p.bias[tr.sigma]);
    const float *ws = tr.sigma ? p.w_scale[1] : p.w_scale[0];
    const float asc = p.a_scale[tr.row0 + min(rl, tr.nrows - 1)];
    float v[TN][4];
    float am0 = 0.f, am1 = 0.f;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int nc = cbase + j * 16;
      const uint2 bu = *reinterpret_cast<const uint2 *>(bias + nc);
      const float4 wsc = *reinterpret_cast<const float4 *>(ws + nc);
      const float b[4] = {__uint_as_float(bu.x << 16), __uint_as_float(bu.x & 0xffff0000u),
                          __uint_as_float(bu.y << 16), __uint_as_float(bu.y & 0xffff0000u)};
      v[j][0] = acc[j][0] * (asc * wsc.x) + b[0];
      v[j][1] = acc[j][1] * (asc * wsc.y) + b[1];
      v[j][2] = acc[j][2] * (asc * wsc.z) + b[2];
      v[j][3] = acc[j][3] * (asc * wsc.w) + b[3];
      const float m = fmaxf(fmaxf(fabsf(v[j][0]), fabsf(v[j][1])), fmaxf(fabsf(v[j][2]), fabsf(v[j][3])));
      if (j / jph == 0) am0 = fmaxf(am0, m);
      else am1 = fmaxf(am1, m);
    }
    am0 = fmaxf(am0, __shfl_xor(am0, 16, 64));
    am0 = fmaxf(am0, __shfl_xor(am0, 32, 64));
    am1 = fmaxf(am1, __shfl_xor(am1, 16, 64));
    am1 = fmaxf(am1, __shfl_xor(am1, 32, 64));
    const int k0 = pow2_exponent(am0), k1 = pow2_exponent(am1);
    const float inv0 = pow2_inverse(k0), inv1 = pow2_inverse(k1);
    if (rl >= tr.nrows) return;
    uint8_t *row = p.qk8 + size_t(tr.row0 + rl) * p.ldq8;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const float s = j / jph == 0 ? inv0 : inv1;
      *reinterpret_cast<uint32_t *>(row + cbase + j * 16) = fp8x4(v[j][0] * s, v[j][1] * s, v[j][2] * s, v[j][3] * s);
    }
    if ((lane >> 4) == 0) {
      row[2 * p.D + wc0 / hd] = uint8_t(127 + k0);
      if (jph * 2 == TN) row[2 * p.D + wc0 / hd + 1] = uint8_t(127 + k1);
    }
  }

  // Epilogue of fragment row i0 of wave wid (each fragment: 4 consecutive columns of one row).  Loads use
  // indices clamped into the tile; values for rows or columns outside it are never stored.
  template <int EPI, bool F8>
  HILO_DEV static void epilogue_row(const GemmProblem &p, const TileRows &tr, int n0, int wid, int i0, int lane,
                                    const f32x4 (&acc)[TN]) {
    const int rl = (wid / WN) * (BM / WM) + i0 * 16 + (lane & 15);
    const int cbase = n0 + (wid % WN) * (BN / WN) + CL * (lane >> 4);
    const size_t m = size_t(tr.row0 + min(rl, tr.nrows - 1));
    const uint16_t *bias = reinterpret_cast<const uint16_t *>(p.bias[tr.sigma]);
    float bv[TN][4];
    float4 gt[TN], zv[TN], wsc[TN];
    float asc;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int nc = min(cbase + j * CS, p.N - 4);
      const uint2 bu = *reinterpret_cast<const uint2 *>(bias + nc);
      bv[j][0] = __uint_as_float(bu.x << 16); bv[j][1] = __uint_as_float(bu.x & 0xffff0000u);
      bv[j][2] = __uint_as_float(bu.y << 16); bv[j][3] = __uint_as_float(bu.y & 0xffff0000u);
      if constexpr (EPI == EPI_RESID) {
        gt[j] = *reinterpret_cast<const float4 *>(p.mod + (size_t(tr.s * 2 + tr.sigma) * 6 + p.gate_idx) * p.D + nc);
        zv[j] = *reinterpret_cast<const float4 *>(p.z + m * p.ldz + nc);
      }
      if constexpr (F8) wsc[j] = *reinterpret_cast<const float4 *>((tr.sigma ? p.w_scale[1] : p.w_scale[0]) + nc);
    }
    if constexpr (F8) asc = p.a_scale[m];
    if (rl >= tr.nrows) return;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int n = cbase + j * CS;
      if (n >= p.N) continue;
      float v[4];
      if constexpr (F8) {
        v[0] = acc[j][0] * (asc * wsc[j].x) + bv[j][0];
        v[1] = acc[j][1] * (asc * wsc[j].y) + bv[j][1];
        v[2] = acc[j][2] * (asc * wsc[j].z) + bv[j][2];
        v[3] = acc[j][3] * (asc * wsc[j].w) + bv[j][3];
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = acc[j][e] + bv[j][e];
      }
      if constexpr (EPI == EPI_RESID) {
        float4 zn = zv[j];
        zn.x += gt[j].x * v[0];
        zn.y += gt[j].y * v[1];
        zn.z += gt[j].z * v[2];
        zn.w += gt[j].w * v[3];
        *reinterpret_cast<float4 *>(p.z + m * p.ldz + n) = zn;
      } else {
        if constexpr (EPI == EPI_GELU) {
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = gelu_tanh(v[e]);
        }
        uint2 u;
        u.x = pack_bf16x2(v[0], v[1]);
        u.y = pack_bf16x2(v[2], v[3]);
        *reinterpret_cast<uint2 *>(reinterpret_cast<uint16_t *>(p.out) + m * p.ldo + n) = u;
      }
    }
  }
};

// Values that are the same on every lane, restated as such (the compiler otherwise keeps some of
// the stream-K bookkeeping in VGPRs and branches on it with exec masks).
HILO_DEV int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
HILO_DEV float *uni(float *ptr) {
  const uint64_t v = reinterpret_cast<uint64_t>(ptr);
  const uint32_t lo = __builtin_amdgcn_readfirstlane(uint32_t(v)), hi = __builtin_amdgcn_readfirstlane(uint32_t(v >> 32));
  return reinterpret_cast<float *>((uint64_t(hi) << 32) | lo);
}
HILO_DEV SkItem uni(const SkItem &x) { return SkItem{uni(x.t), uni(x.kb), uni(x.ke), uni(x.slot), uni(int(x.valid)) != 0}; }
HILO_DEV TileRows uni(const TileRows &x) { return TileRows{uni(x.s), uni(x.sigma), uni(x.row0), uni(x.nrows)}; }

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef int i32x8 __attribute__((ext_vector_type(8)));

// One 4-byte global load per lane straight into LDS: lane l lands at byte 4 l of the destination.
HILO_DEV void g2lds4(const void *g, void *lds_wave_base) {
  __builtin_amdgcn_global_load_lds(g, (__attribute__((address_space(3))) void *)lds_wave_base, 4, 0, 0);
}

// ----------------------------------------------------------- bf16 and FP8 tiles on eight waves
//
// One persistent workgroup of 8 waves per CU (2 x 4: wave tile BM/2 x BN/4 as 16 x 16 MFMA blocks, two
// waves per SIMD).  A K step is a window of 64 values, 128-byte rows of A and W; LDS holds SLOTS windows
// filled by direct global->LDS loads of 8 whole lines each (16-byte chunk c of row r at c ^ (r / 2) % 8,
// so that the 16 rows a fragment read touches fall on 16 bank groups, natural or permuted order alike).
// A window is two halves of 32 values; while the MFMAs of one half run, the fragments of the next are
// read into the other register set, a few between the rows of blocks, so the matrix core of a SIMD waits
// for LDS only where both of its waves do.  One barrier per window, between its halves: by then every
// wave has read the window (its slot is refilled during the second half) and the next window has landed.
//
// What bounds it: the matrix core at the clock the power limit leaves (MFMAs alone 2.05 PFLOP/s on
// random data), the fragment reads and the L2-to-LDS path in about equal parts -- without the reads or
// without the loads the 256 x 256 loop runs 12-15% faster, without either 30%.  A CU takes in ~120 GB/s
// of L2 hits and ~30 GB/s of misses, so the bytes per FLOP of the tile matter: 23040 x 12288 x 3072 runs
// 1247 us on 256 x 256 tiles (1.40 PFLOP/s), 1391 on 192 x 192; the 4-wave loop before took ~1750 (192 x
// 192, one wave per SIMD: every memory instruction held its only MFMA stream).  Two 4-wave groups in
// ping-pong (one in its MFMAs, the other reading) ran 1370 and 1347 us; 32 x 32 MFMAs in this schedule
// 1367; s_setprio around the MFMAs cost 1%.
//
// FP8: a window holds 128 values, and an FP8 MFMA takes the same cycles per operand byte as a bf16 one, so
// the loads, reads and MFMA time per window are those of bf16.  256 x 256 tiles: v_mfma_f32_32x32x64_f8f6f4
// per half (16 x 16 x 128 fragments of 32 bytes a lane would not fit twice), on 4 x 2 waves so that a wave
// holds whole heads.  192 x 192 tiles: v_mfma_f32_16x16x128_f8f6f4 per window (the wave's 96 x 48 is not
// whole 32 x 32 blocks).  Against one wave per SIMD the 64 x 64 step with the FP8 block went 597 -> 577 us; the
// MLP half on 7680 rows is level (689 and 684, noise 0.3% and more between boxes).
namespace g8 {
// A BM x BN tile of bf16 or FP8 operands on 8 waves: WM x WN waves, MB x NB blocks of 16 x 16 each (B32: of
// 32 x 32).
template <int BM, int BN, bool F8 = false>
struct Geo {
  static constexpr bool B32 = F8 && BN == 256;
  static constexpr int WN = B32 ? 2 : 4, WM = 8 / WN;
  static constexpr int MB = BM / WM / (B32 ? 32 : 16), NB = BN / WN / (B32 ? 32 : 16);
  static constexpr int LA = BM / 64, LB = BN / 64;  // load instructions per wave and window
  static constexpr int WB = (BM + BN) * 128;        // bytes of a window
  static constexpr int KW = F8 ? 128 : 64;          // values of K in a window
  // per wave, behind the windows: its columns of bias (bf16), of the gate (float32) and, for FP8, of the
  // weight scales and its rows of activation scales (float32)
  static constexpr int kGate = 256, kCol = 512, kRow = 1024, kEpi = F8 ? 1536 : 512;
  static constexpr int SLOTS = 3 * WB + 8 * kEpi <= 160 * 1024 ? 3 : 2;
  static constexpr int LDS = SLOTS * WB + 8 * kEpi;
};
// Chunk swizzle of window rows; B32 reads W rows in the order perm_w, whose 16-lane groups (rows 0-3, 16-19,
// 4-7, 20-23, ...) need bit 4 in it to fall on 16 bank groups.
template <bool B32>
HILO_DEV int swz(int r) {
  if constexpr (B32) return ((r >> 1) & 3) ^ ((((r >> 3) ^ (r >> 4)) & 1) << 2);
  else return (r >> 1) & 7;
}
// W row read by fragment lane r of a 32 x 32 block.  The MFMA's output row i (the W side) lands in
// accumulator register 4 (i / 8) + i % 4 of the lanes of half (i / 4) % 2; reading W row perm_w(i) there
// gives lane half g the columns 16 g .. 16 g + 15 in register order.
HILO_DEV int perm_w(int r) { return ((r & 4) ? 16 : 0) + 4 * (r >> 3) + (r & 3); }
template <int V>
struct Int {
  static constexpr int value = V;
};
template <int N>
HILO_DEV void wait_vm() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }
HILO_DEV i32x8 cat8(u32x4 lo, u32x4 hi) {
  return __builtin_bit_cast(i32x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}
}  // namespace g8

template <int OFF, typename V>
HILO_DEV void ds_read16(V &d, uint32_t addr) {
  static_assert(sizeof(V) == 16);
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(d) : "v"(addr), "n"(OFF) : "memory");
}

// FP8 tiles of 32 x 32 blocks (256 x 256, the wave's 64 x 128): lane l of block (bi, bj) holds row 32 bi +
// l % 32 and columns 32 bj + 16 (l / 32) .. + 15 in register order.  The 16 values acc * (row scale * weight
// scale) + bias of a block, operands from the wave's LDS area.
template <typename G>
HILO_DEV void values32(const uint8_t *epi, int lane, int bj, float sa, const f32x16 &blk, float (&v)[16]) {
  const int cl = 16 * (lane >> 5) + 32 * bj;
  u32x4 bu[2];
  f32x4 cv[4];
#pragma unroll
  for (int h = 0; h < 2; ++h) bu[h] = *reinterpret_cast<const u32x4 *>(epi + 2 * cl + 16 * h);
#pragma unroll
  for (int h = 0; h < 4; ++h) cv[h] = *reinterpret_cast<const f32x4 *>(epi + G::kCol + 4 * cl + 16 * h);
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const uint32_t w = bu[e >> 3][(e >> 1) & 3];
    const float bias = __uint_as_float((e & 1) ? (w & 0xffff0000u) : (w << 16));
    v[e] = blk[e] * (sa * cv[e >> 2][e & 3]) + bias;
  }
}

template <typename G>
HILO_DEV void epilogue32(const GemmProblem &p, const TileRows &tr, int n0, int wm, int lane, const uint8_t *epi,
                         f32x16 (&acc)[G::MB][G::NB]) {
#pragma unroll
  for (int bi = 0; bi < G::MB; ++bi) {
    const int rl = (wm * G::MB + bi) * 32 + (lane & 31);
    const float sa = *reinterpret_cast<const float *>(epi + G::kRow + 4 * (32 * bi + (lane & 31)));
#pragma unroll
    for (int bj = 0; bj < G::NB; ++bj) {
      const int n = n0 + 32 * bj + 16 * (lane >> 5);
      if (rl < tr.nrows && n < p.N) {  // N % 16 == 0: a lane's 16 columns are all inside or all out
        float v[16];
        values32<G>(epi, lane, bj, sa, acc[bi][bj], v);
        uint4 *op = reinterpret_cast<uint4 *>(reinterpret_cast<uint16_t *>(p.out) + size_t(tr.row0 + rl) * p.ldo + n);
#pragma unroll
        for (int h = 0; h < 2; ++h)
          op[h] = make_uint4(pack_bf16x2(v[8 * h + 0], v[8 * h + 1]), pack_bf16x2(v[8 * h + 2], v[8 * h + 3]),
                             pack_bf16x2(v[8 * h + 4], v[8 * h + 5]), pack_bf16x2(v[8 * h + 6], v[8 * h + 7]));
      }
      asm volatile("" ::: "memory");  // the next block's operands stay below these stores
    }
  }
}

// FP8 q and k for the attention's score product, of a tile whose columns lie below 2 D.  The wave's 128
// columns hold whole heads (128 / head_dim of them); per (row, head): the amax of the values over the head
// -- this lane's 16 columns of each block and those of lane l ^ 32, which holds the block's other 16 -- the
// power-of-two scale 2^k, the E4M3 codes of the values times 2^-k (16 bytes per lane and block) and one
// E8M0 byte 127 + k.  The values are formed twice (amax, then codes) instead of held.
template <typename G>
HILO_DEV void epilogue32_qk8(const GemmProblem &p, const TileRows &tr, int n0, int wm, int lane, const uint8_t *epi,
                             f32x16 (&acc)[G::MB][G::NB]) {
  const int hd = p.head_dim, bph = hd / 32;  // blocks per head
#pragma unroll
  for (int bi = 0; bi < G::MB; ++bi) {
    const float sa = *reinterpret_cast<const float *>(epi + G::kRow + 4 * (32 * bi + (lane & 31)));
    float am0 = 0.f, am1 = 0.f;
#pragma unroll
    for (int bj = 0; bj < G::NB; ++bj) {
      float v[16];
      values32<G>(epi, lane, bj, sa, acc[bi][bj], v);
      float m = 0.f;
#pragma unroll
      for (int e = 0; e < 16; ++e) m = fmaxf(m, fabsf(v[e]));
      if (bj / bph == 0) am0 = fmaxf(am0, m);
      else am1 = fmaxf(am1, m);
    }
    am0 = fmaxf(am0, __shfl_xor(am0, 32, 64));
    am1 = fmaxf(am1, __shfl_xor(am1, 32, 64));
    const int k0 = pow2_exponent(am0), k1 = pow2_exponent(am1);
    const float i0 = pow2_inverse(k0), i1 = pow2_inverse(k1);
    const int rl = (wm * G::MB + bi) * 32 + (lane & 31);
    if (rl < tr.nrows) {
      uint8_t *row = p.qk8 + size_t(tr.row0 + rl) * p.ldq8;
#pragma unroll
      for (int bj = 0; bj < G::NB; ++bj) {
        float v[16];
        values32<G>(epi, lane, bj, sa, acc[bi][bj], v);
        const float s = bj / bph == 0 ? i0 : i1;
        uint4 c;
        c.x = fp8x4(v[0] * s, v[1] * s, v[2] * s, v[3] * s);
        c.y = fp8x4(v[4] * s, v[5] * s, v[6] * s, v[7] * s);
        c.z = fp8x4(v[8] * s, v[9] * s, v[10] * s, v[11] * s);
        c.w = fp8x4(v[12] * s, v[13] * s, v[14] * s, v[15] * s);
        *reinterpret_cast<uint4 *>(row + n0 + 16 * (lane >> 5) + 32 * bj) = c;
      }
      if (lane < 32) {
        row[2 * p.D + n0 / hd] = uint8_t(127 + k0);
        if (bph * 2 == G::NB) row[2 * p.D + n0 / hd + 1] = uint8_t(127 + k1);
      }
    }
    asm volatile("" ::: "memory");
  }
}

// All work items of this workgroup under plan q on BM x BN tiles.
template <int BM, int BN, int EPI, bool F8 = false>
HILO_DEV void gemm8_run(const GemmProblem &p, const SkPlan &q, int pid, uint8_t *lds) {
  using namespace g8;
  using G = Geo<BM, BN, F8>;
  constexpr bool B32 = G::B32;
  using T = SkTile<BM, BN, G::WM, G::WN, !B32>;
  constexpr int MB = G::MB, NB = G::NB, LA = G::LA, LB = G::LB, WB = G::WB, S = G::SLOTS;
  constexpr int WM = G::WM, WN = G::WN, ESZ = F8 ? 1 : 2;  // ESZ: operand bytes per element
  const int lane = threadIdx.x & 63;
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lr = lane & 15, lg = lane >> 4, wm = wid / WN, wn = wid % WN;
  const SkRange rg = sk_range(q, pid);

  // ---- loader: its own cursor over the items, S windows ahead of the MFMAs; wave wid loads rows
  // wid BM/8 .. of A and wid BN/8 .. of W, 8 rows per instruction: a uniform base plus a lane offset
  SkCursor lc{pid, rg.beg};
  const char *la = nullptr, *lb = nullptr;
  uint32_t oa[LA], ob[LB];
  int lk = 0, lke = 0, lslot = 0;
  auto ld_advance = [&]() __attribute__((always_inline)) {
    const SkItem x = uni(sk_next_item(lc, q, rg, pid, p.part, T::kPartFloats));
    if (!x.valid) {  // no further item: repeat the last window (its slots are free, its addresses valid)
      --lk;
      la -= 128;
      lb -= 128;
      return;
    }
    int rt, tn;
    tile_coords(q, x.t, rt, tn);
    const TileRows tr = uni(decode_row_tile(p, BM, uni(rt)));
    const int n0 = uni(tn) * BN;
    const int lane = opaque(threadIdx.x & 63);
#pragma unroll
    for (int i = 0; i < LA; ++i) {
      const int r = wid * (BM / 8) + 8 * i + (lane >> 3);
      oa[i] = uint32_t(min(r, tr.nrows - 1)) * uint32_t(p.lda) * ESZ + uint32_t((lane & 7) ^ swz<B32>(r)) * 16;
    }
#pragma unroll
    for (int i = 0; i < LB; ++i) {
      const int r = wid * (BN / 8) + 8 * i + (lane >> 3);
      ob[i] = uint32_t(min(r, p.N - 1 - n0)) * uint32_t(p.K) * ESZ + uint32_t((lane & 7) ^ swz<B32>(r)) * 16;
    }
    la = reinterpret_cast<const char *>(p.A) + (size_t(tr.row0) * p.lda + size_t(x.kb) * G::KW) * ESZ;
    lb = reinterpret_cast<const char *>(tr.sigma ? p.W[1] : p.W[0]) + (size_t(n0) * p.K + size_t(x.kb) * G::KW) * ESZ;
    lk = x.kb;
    lke = x.ke;
  };
  auto ld_a = [&]() __attribute__((always_inline)) {
    uint8_t *d = lds + lslot * WB + wid * (BM / 8) * 128;
#pragma unroll
    for (int i = 0; i < LA; ++i) g2lds16(la + oa[i], d + i * 1024);
    la += 128;
  };
  auto ld_b = [&]() __attribute__((always_inline)) {
    uint8_t *d = lds + lslot * WB + (BM + wid * (BN / 8)) * 128;
#pragma unroll
    for (int i = 0; i < LB; ++i) g2lds16(lb + ob[i], d + i * 1024);
    lb += 128;
    ++lk;
    lslot = lslot == S - 1 ? 0 : lslot + 1;
  };

  // ---- fragments, in chunks of 16 bytes.  bf16: lane (lr, lg) holds chunk 4 h + lg of row lr of a 16-row
  // block in half h.  FP8, 16 x 16 blocks: both of these at once, for one 128-deep MFMA.  FP8, 32 x 32
  // blocks: chunks 4 h + g and 4 h + 2 + g (g = lane / 32) of row lane % 32 for one 64-deep MFMA of half h.
  // W rows of 16 x 16 blocks go in the order that gives the lane's accumulators 4 NB consecutive columns:
  // MFMA output row 4 g + e of block j is column 4 NB g + 4 j + e of the wave
  constexpr int NC = F8 ? 2 : 1;                       // chunks of a fragment
  constexpr int NR = (MB + NB) * NC;                   // reads of a set: W first, then A
  constexpr int NA = B32 ? 4 : 2;                      // chunk addresses of a lane
  constexpr int RB = B32 ? 4096 : 2048;                // bytes between blocks
  using Acc = std::conditional_t<B32, f32x16, f32x4>;
  using Frag = std::conditional_t<F8, u32x4, bf16x8>;
  const uint32_t lds0 = (uint32_t)(uintptr_t)lds;
  uint32_t fa[NA], fb[B32 ? 1 : NB][NA];
#pragma unroll
  for (int h = 0; h < NA; ++h) {
    if constexpr (B32) {
      const int r = lane & 31, w = perm_w(r), c = 2 * h + (lane >> 5);
      fa[h] = lds0 + (wm * (BM / WM) + r) * 128 + ((c ^ swz<B32>(r)) * 16);
      fb[0][h] = lds0 + (BM + wn * (BN / WN) + w) * 128 + ((c ^ swz<B32>(w)) * 16);
    } else {
      fa[h] = lds0 + (wm * (BM / WM) + lr) * 128 + (((4 * h + lg) ^ swz<B32>(lr)) * 16);
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const int r = wn * (BN / WN) + (lr >> 2) * 4 * NB + 4 * j + (lr & 3);
        fb[j][h] = lds0 + (BM + r) * 128 + (((4 * h + lg) ^ swz<B32>(r)) * 16);
      }
    }
  }
  Acc acc[MB][NB];
  // Two sets: the halves of a window, or (FP8, 16 x 16) two windows.  The latter has no registers for two
  // whole sets: rows 0 .. MB - 3 of A keep one fragment each, re-read once the row's MFMAs are issued
  Frag a[2][MB][NC], b[2][NB][NC];
  constexpr bool INP = F8 && !B32;
  auto set_a = [](int h, int i) constexpr { return INP && i < MB - 2 ? 0 : h; };
  uint32_t so = 0;  // byte offset of the window being read
  // read x of set h
  auto rd = [&](auto hh, auto xx) __attribute__((always_inline)) {
    constexpr int h = decltype(hh)::value, x = decltype(xx)::value / NC, c = decltype(xx)::value % NC;
    constexpr int ad = B32 ? 2 * h + c : F8 ? c : h;
    if constexpr (x < NB) {
      if constexpr (B32) ds_read16<(x < NB ? x : 0) * RB>(b[h][x][c], fb[0][ad] + so);
      else ds_read16<0>(b[h][x][c], fb[x][ad] + so);
    } else if constexpr (x < NB + MB) {
      ds_read16<(x - NB) * RB>(a[set_a(h, x - NB)][x - NB][c], fa[ad] + so);
    }
  };
  auto rd_wait = [&](auto hh) __attribute__((always_inline)) {
    constexpr int h = decltype(hh)::value;
    // lgkmcnt(0), in the form the compiler's own wait tracking sees
    __builtin_amdgcn_s_waitcnt(0xc07f);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
#pragma unroll
      for (int i = 0; i < MB; ++i) asm volatile("" : "+v"(a[set_a(h, i)][i][c]));
#pragma unroll
      for (int j = 0; j < NB; ++j) asm volatile("" : "+v"(b[h][j][c]));
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  auto rd_all = [&](auto hh) __attribute__((always_inline)) {
    auto r6 = [&](auto x) __attribute__((always_inline)) {
      constexpr int x0 = decltype(x)::value;
      if constexpr (x0 < NR) {
        rd(hh, Int<x0>{}); rd(hh, Int<x0 + 1>{}); rd(hh, Int<x0 + 2>{});
        rd(hh, Int<x0 + 3>{}); rd(hh, Int<x0 + 4>{}); rd(hh, Int<x0 + 5>{});
      }
    };
    static_assert(NR <= 18, "reads of a set");
    r6(Int<0>{}); r6(Int<6>{}); r6(Int<12>{});
    rd_wait(hh);
  };
  // the MFMAs of set h in MB (B32: MB NB) groups; after each group a share of the reads of the other set,
  // and (ld) the loads of a window into the slot just freed
  auto half = [&](auto hh, auto ldd) __attribute__((always_inline)) {
    constexpr int h = decltype(hh)::value;
    constexpr int GR = B32 ? MB * NB : MB;
    constexpr int RPB = B32 || INP ? 2 : (NR + MB - 2) / (MB - 1);  // reads per group, none after the last
    static_assert(RPB == 2, "reads per group of MFMAs");
    auto row = [&](auto ii) __attribute__((always_inline)) {
      constexpr int i = decltype(ii)::value;
      if constexpr (i < GR) {
        if constexpr (B32) {
          acc[i / NB][i % NB] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
              cat8(b[h][i % NB][0], b[h][i % NB][1]), cat8(a[h][i / NB][0], a[h][i / NB][1]), acc[i / NB][i % NB], 0, 0,
              0, 0, 0, 0);
        } else {
#pragma unroll
          for (int j = 0; j < NB; ++j) {
            if constexpr (F8)
              acc[i][j] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(
                  cat8(b[h][j][0], b[h][j][1]), cat8(a[set_a(h, i)][i][0], a[set_a(h, i)][i][1]), acc[i][j], 0, 0, 0, 0, 0,
                  0);
            else
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[h][j][0], a[h][i][0], acc[i][j], 0, 0, 0);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (INP) {
          // after row i: A fragment i; W 0 and 1 after row 0, 2 after row 1, A MB - 2 and MB - 1 after 2 and 3
          static_assert(MB == 6 && NB == 3, "read order of the FP8 tile");
          if constexpr (i < 2) {
            rd(Int<1 - h>{}, Int<4 * i>{});
            rd(Int<1 - h>{}, Int<4 * i + 1>{});
          }
          if constexpr (i == 0) {
            rd(Int<1 - h>{}, Int<2>{});
            rd(Int<1 - h>{}, Int<3>{});
          }
          if constexpr (i < MB - 2) {
            rd(Int<1 - h>{}, Int<2 * (NB + i)>{});
            rd(Int<1 - h>{}, Int<2 * (NB + i) + 1>{});
          }
          if constexpr (i == 2 || i == 3) {
            rd(Int<1 - h>{}, Int<2 * (NB + i + 2)>{});
            rd(Int<1 - h>{}, Int<2 * (NB + i + 2) + 1>{});
          }
        } else {
          rd(Int<1 - h>{}, Int<i * RPB>{});
          rd(Int<1 - h>{}, Int<i * RPB + 1>{});
        }
        if constexpr (decltype(ldd)::value) {
          if constexpr (i == 0) ld_a();
          if constexpr (i == GR / 2) ld_b();
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    row(Int<0>{}); row(Int<1>{}); row(Int<2>{}); row(Int<3>{});
    row(Int<4>{}); row(Int<5>{}); row(Int<6>{}); row(Int<7>{});
  };
  // this wave has read the window; all but the last window issued have landed (the epilogue's DMA, issued
  // behind that one, only makes this wait stricter); on to the next
  auto next_window = [&]() __attribute__((always_inline)) {
    wait_vm<(S - 2) * (LA + LB)>();
    asm volatile("s_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    so = so == (S - 1) * WB ? 0 : so + WB;
    if (lk == lke) ld_advance();
  };

  // ---- epilogue operands of the current item: the wave's columns of bias, gate and scales, by DMA
  uint8_t *epi = lds + S * WB + wid * G::kEpi;
  SkCursor cc{pid, rg.beg};
  SkItem cur = uni(sk_next_item(cc, q, rg, pid, p.part, T::kPartFloats));
  if (!cur.valid) return;
  ld_advance();  // the same first item
#pragma unroll 1
  for (int w = 0; w < S; ++w) {
    if (lk == lke) ld_advance();
    ld_a();
    ld_b();
  }
  wait_vm<(S - 1) * (LA + LB)>();
  asm volatile("s_barrier" ::: "memory");
  TileRows etr{0, 0, 0, 1};
  int en0 = 0;
  while (true) {
    const bool whole = cur.slot == nullptr;
    if (whole) {
      int rt, tn;
      tile_coords(q, cur.t, rt, tn);
      en0 = uni(tn) * BN + wn * (BN / WN);
      etr = uni(decode_row_tile(p, BM, uni(rt)));
      const uint16_t *bias = reinterpret_cast<const uint16_t *>(etr.sigma ? p.bias[1] : p.bias[0]);
      g2lds4(bias + min(en0 + 2 * lane, p.N - 2), epi);
      if constexpr (EPI == EPI_RESID)
        g2lds4(p.mod + (size_t(etr.s * 2 + etr.sigma) * 6 + p.gate_idx) * p.D + min(en0 + lane, p.N - 1), epi + G::kGate);
      if constexpr (F8) {
        const float *ws = etr.sigma ? p.w_scale[1] : p.w_scale[0];
        const int r0 = wm * (BM / WM);
        g2lds4(ws + min(en0 + lane, p.N - 1), epi + G::kCol);
        if constexpr (BN / WN > 64) g2lds4(ws + min(en0 + 64 + lane, p.N - 1), epi + G::kCol + 256);
        g2lds4(p.a_scale + etr.row0 + min(r0 + lane, etr.nrows - 1), epi + G::kRow);
        if constexpr (BM / WM > 64) g2lds4(p.a_scale + etr.row0 + min(r0 + 64 + lane, etr.nrows - 1), epi + G::kRow + 256);
      }
    }
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j) acc[i][j] = Acc(0.f);
    // the first window's first fragments (again, after an epilogue: it needs their registers)
    rd_all(Int<0>{});
    if constexpr (INP) {
      int kt = cur.kb;
#pragma unroll 1
      for (; kt + 1 < cur.ke; kt += 2) {
        next_window();
        half(Int<0>{}, std::true_type{});
        rd_wait(Int<1>{});
        next_window();
        half(Int<1>{}, std::true_type{});
        rd_wait(Int<0>{});
      }
      if (kt < cur.ke) {
        next_window();
        half(Int<0>{}, std::true_type{});
        rd_wait(Int<1>{});
      }
    } else {
#pragma unroll 1
      for (int kt = cur.kb; kt < cur.ke; ++kt) {
        half(Int<0>{}, std::false_type{});
        rd_wait(Int<1>{});
        next_window();
        half(Int<1>{}, std::true_type{});
        rd_wait(Int<0>{});
      }
    }
    if (whole) {
      // a one-step item's epilogue operands may still be in flight
      if (cur.ke - cur.kb < 2) wait_vm<0>();
    }
    const int lane = opaque(threadIdx.x & 63), lr = lane & 15, lg = lane >> 4;
    if constexpr (B32) {
      static_assert(EPI != EPI_RESID && EPI != EPI_GELU, "epilogues of 32 x 32 blocks");
      if (whole) {
        if (p.qk8 != nullptr && en0 < 2 * p.D) epilogue32_qk8<G>(p, etr, en0, wm, lane, epi, acc);
        else epilogue32<G>(p, etr, en0, wm, lane, epi, acc);
      } else {
        // the fixup's 16 x 16 order: row 32 bi + l % 32 is fragment row 2 bi + (l % 32) / 16; columns 32 bj
        // + 16 (l / 32) + 4 c .. + 3 are lane l % 16 + 16 c of fragment column 2 bj + l / 32
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
          for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int c = 0; c < 4; ++c)
              *reinterpret_cast<f32x4 *>(cur.slot + T::part_index(wid, 2 * i + ((lane & 31) >> 4), 2 * j + (lane >> 5),
                                                                  lr + 16 * c)) =
                  f32x4{acc[i][j][4 * c], acc[i][j][4 * c + 1], acc[i][j][4 * c + 2], acc[i][j][4 * c + 3]};
      }
    } else if (whole) {
      uint2 bu[NB];
      f32x4 wsc[F8 ? NB : 1];
      f32x4 gv[NB];
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        bu[j] = *reinterpret_cast<const uint2 *>(epi + 2 * (4 * NB * lg + 4 * j));
        if constexpr (EPI == EPI_RESID) gv[j] = *reinterpret_cast<const f32x4 *>(epi + G::kGate + 4 * (4 * NB * lg + 4 * j));
        if constexpr (F8) wsc[j] = *reinterpret_cast<const f32x4 *>(epi + G::kCol + 4 * (4 * NB * lg + 4 * j));
      }
      const int nc = en0 + 4 * NB * lg;
      // the residual update keeps the z pieces of ZS batches of two row blocks in flight: stores count in
      // vmcnt, so a load issued behind them waits for them too.  Two batches of a 256 x 256 tile are 64
      // registers beside its 128 accumulators, a third would not fit (64 registers went to scratch, whose
      // accesses wait for each other and for the loads in flight); on 192 x 192 three are the whole tile.
      // 25004 rows in 8 samples: output 559 -> 515 us, MLP down 1661 -> 1600 against the three that spilled.
      constexpr int ZR = EPI == EPI_RESID ? 2 : 1, ZS = NB == 4 ? 2 : 3;
      static_assert(MB % ZR == 0, "row blocks per batch");
      f32x4 z[ZS][ZR][NB];
      // z is addressed by 32-bit offsets from the tile's first row (at most 256 rows of 8192 values)
      char *zt = reinterpret_cast<char *>(p.z + size_t(etr.row0) * p.ldz);
      auto zoff = [&](int r, int j) __attribute__((always_inline)) {
        // N % 64 == 0: a lane's 16 columns of a 256-wide tile are all inside or all out
        const int n = NB == 4 ? min(nc, p.N - 16) + 4 * j : min(nc + 4 * j, p.N - 4);
        return (uint32_t(r) * uint32_t(p.ldz) + uint32_t(n)) * 4;
      };
      auto ld_z = [&](int set, int i0) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < ZR; ++i) {
          const int rl = wm * (BM / WM) + 16 * (i0 + i) + lr;
#pragma unroll
          for (int j = 0; j < NB; ++j) z[set][i][j] = *reinterpret_cast<const f32x4 *>(zt + zoff(min(rl, etr.nrows - 1), j));
        }
      };
      if constexpr (EPI == EPI_RESID) {
#pragma unroll
        for (int s = 0; s < ZS; ++s)
          if (s * ZR < MB) ld_z(s, s * ZR);
      }
#pragma unroll
      for (int i0 = 0; i0 < MB; i0 += ZR) {
#pragma unroll
        for (int ii = 0; ii < ZR; ++ii) {
          const int i = i0 + ii, rl = wm * (BM / WM) + 16 * i + lr;
          // taken here whether used or not: a load still pending at the K loop would put a vmcnt(0) into it
          if constexpr (EPI == EPI_RESID) {
#pragma unroll
            for (int j = 0; j < NB; ++j) asm volatile("" : "+v"(z[i0 / ZR % ZS][ii][j]));
          }
          if (rl < etr.nrows) {
            const size_t m = size_t(etr.row0 + rl);
            uint2 o[NB];
            float sa;
            if constexpr (F8) sa = *reinterpret_cast<const float *>(epi + G::kRow + 4 * (16 * i + lr));
#pragma unroll
            for (int j = 0; j < NB; ++j) {
              float v[4];
              const float bv[4] = {__uint_as_float(bu[j].x << 16), __uint_as_float(bu[j].x & 0xffff0000u),
                                   __uint_as_float(bu[j].y << 16), __uint_as_float(bu[j].y & 0xffff0000u)};
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                if constexpr (F8) v[e] = acc[i][j][e] * (sa * wsc[j][e]) + bv[e];
                else v[e] = acc[i][j][e] + bv[e];
              }
              if constexpr (EPI == EPI_RESID) {
                f32x4 zn = z[i0 / ZR % ZS][ii][j];
#pragma unroll
                for (int e = 0; e < 4; ++e) zn[e] += gv[j][e] * v[e];
                if (nc + 4 * j < p.N) *reinterpret_cast<f32x4 *>(zt + zoff(rl, j)) = zn;
              } else {
                if constexpr (EPI == EPI_GELU) {
#pragma unroll
                  for (int e = 0; e < 4; ++e) v[e] = gelu_tanh(v[e]);
                }
                o[j] = make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
              }
            }
            if constexpr (EPI != EPI_RESID) {
              uint16_t *op = reinterpret_cast<uint16_t *>(p.out) + m * p.ldo + nc;
#pragma unroll
              for (int j = 0; j < NB; ++j)
                if (nc + 4 * j < p.N) *reinterpret_cast<uint2 *>(op + 4 * j) = o[j];
            }
          }
        }
        asm volatile("" ::: "memory");  // the next blocks' operands stay below these stores
        if constexpr (EPI == EPI_RESID) {
          if (i0 + ZS * ZR < MB) ld_z(i0 / ZR % ZS, i0 + ZS * ZR);
        }
      }
    } else {
      float *slot = cur.slot;
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) *reinterpret_cast<f32x4 *>(slot + T::part_index(wid, i, j, lane)) = acc[i][j];
    }
    cur = uni(sk_next_item(cc, q, rg, pid, p.part, T::kPartFloats));
    if (!cur.valid) break;
  }
  wait_vm<0>();
}

// Small problems: 64 x 32 tiles, four waves each (a workgroup holds two), K split over the four in steps of
// 64 and their sums added through LDS.  Fragments come straight from global memory: lane (lr, lg) takes
// the 32 bytes at 32 lg of a row's 128-byte K step, two chunks for two MFMAs (any order of K will do as
// long as both operands agree).  What bounds it is the latency of one tile, about 3 us plus 1.4 us per
// 256 of K, or 2.65 where both tiles are busy (12 KB of fragments per step and wave at the L2-to-CU rate), so it is the better plan where
// 192 x 192 tiles would leave most CUs idle for a long K: 2 x ~320 rows, D 256, MLP 1024: QKV 14.4 -> 9.1
// us by event pairs, output 20.6 -> 8.1, MLP up 17.2 -> 9.7, MLP down 28.6 -> 12.1; at 704 rows, D 1024, it
// still wins for the output (34.5 -> 18 us) and MLP down (73 -> 49), and loses for QKV (26 against 36).
template <int EPI>
HILO_DEV void gemm_small_run(const GemmProblem &p, int rows, int pid, uint8_t *lds) {
  constexpr int BM = 64, BN = 32, MB = 4, NB = 2;
  f32x4 *part = reinterpret_cast<f32x4 *>(lds);  // [2 tiles][4 waves][8 blocks][64 lanes]
  const int lane = threadIdx.x & 63;
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), w = wid & 3;
  const int lr = lane & 15, lg = lane >> 4;
  const int tilesN = p.N / BN, tiles = rows * tilesN;  // N % 64 == 0
  const int steps = p.K / 64, s0 = steps * w / 4, s1 = steps * (w + 1) / 4;
  for (int t0 = pid; t0 < tiles; t0 += 2 * kGemmWorkgroups) {  // the same number of turns for both tiles
    const int t = t0 + (wid >> 2) * kGemmWorkgroups;
    const bool on = t < tiles;
    const int tn = on ? t % tilesN : 0, n0 = tn * BN;
    const TileRows tr = uni(decode_row_tile(p, BM, on ? t / tilesN : 0));
    const char *A[MB], *W[NB];
#pragma unroll
    for (int i = 0; i < MB; ++i)
      A[i] = reinterpret_cast<const char *>(p.A) + (size_t(tr.row0 + min(16 * i + lr, tr.nrows - 1)) * p.lda) * 2 + 32 * lg;
#pragma unroll
    for (int j = 0; j < NB; ++j)
      W[j] = reinterpret_cast<const char *>(tr.sigma ? p.W[1] : p.W[0]) + (size_t(n0 + 16 * j + lr) * p.K) * 2 + 32 * lg;
    f32x4 acc[MB][NB];
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto load = [&](int s, bf16x8 (&a)[2][MB], bf16x8 (&b)[2][NB]) __attribute__((always_inline)) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int i = 0; i < MB; ++i) a[h][i] = *reinterpret_cast<const bf16x8 *>(A[i] + size_t(s) * 128 + 16 * h);
#pragma unroll
        for (int j = 0; j < NB; ++j) b[h][j] = *reinterpret_cast<const bf16x8 *>(W[j] + size_t(s) * 128 + 16 * h);
      }
    };
    auto mul = [&](const bf16x8 (&a)[2][MB], const bf16x8 (&b)[2][NB]) __attribute__((always_inline)) {
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
          for (int j = 0; j < NB; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[h][j], a[h][i], acc[i][j], 0, 0, 0);
    };
    if (on && s0 < s1) {
      bf16x8 xa[2][MB], xb[2][NB], ya[2][MB], yb[2][NB];
      load(s0, xa, xb);
#pragma unroll 1
      for (int s = s0; s < s1; s += 2) {
        if (s + 1 < s1) load(s + 1, ya, yb);
        mul(xa, xb);
        if (s + 1 >= s1) break;
        if (s + 2 < s1) load(s + 2, xa, xb);
        mul(ya, yb);
      }
    }
    f32x4 *mine = part + (wid * MB * NB) * 64 + lane;
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j) mine[(i * NB + j) * 64] = acc[i][j];
    __syncthreads();
    // wave w finishes row block w: rows 16 w + lr, columns 16 j + 4 lg .. + 3
    if (on && 16 * w + lr < tr.nrows) {
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const f32x4 *src = part + ((wid & 4) * MB * NB + w * NB + j) * 64 + lane;
        const f32x4 v = (src[0] + src[MB * NB * 64]) + (src[2 * MB * NB * 64] + src[3 * MB * NB * 64]);
        const float o[4] = {v[0], v[1], v[2], v[3]};
        epilogue4<EPI, true>(p, tr, tr.row0 + 16 * w + lr, n0 + 16 * j + 4 * lg, o);
      }
    }
    __syncthreads();  // the next tiles' sums go to the same LDS
  }
}

// The tile of a projection, chosen on the device (only it knows the row counts; the main kernel and the
// fixup derive the same one): the shortest of three estimates in units of 10 ns, fitted to forced runs of each
// tile over D 256 .. 4096 and 64 .. 25000 rows (616 projections; the choice loses 0.4% to the best tile on average,
// 1.5% without the terms for a launch and for the number of tiles cut into pieces).  A K step takes 1.46 us on a 256
// x 256 tile and 0.91 on 192 x 192; a tile adds its epilogue, 7 and 4 us, or 33 and 14 where it updates z (every
// workgroup reads and writes its tile's z at once, 26 and 14 us at the copy rate); a launch of whole tiles 7 us (3
// where they update z); a stream-K tail 36 and 20 us for its partials and their fixup.  K pieces spread the K steps
// evenly; their partials, the fixup and z take 45 us and 0.35 a tile, or 27 and 0.2, and 45 or 25 where the pieces of
// T tiles (T a power of two) fill the workgroups without a tail.  A turn of TILE_SMALL takes 1.4 us per four K steps,
// or 2.65 with two tiles a workgroup, and 3.  2766 rows of a 64 x 64 grid: 192 x 192 for all four projections (QKV
// 151 us against 168, output 70 / 108, MLP up 196 / 198, MLP down 188 / 223); 25000 rows in 8 samples: 256 x 256 (QKV
// 1208 against 1256, output 515 / 533, MLP up 1535 / 1660, MLP down 1600 / 1658); D 1536, MLP down at 200 rows: 192 x
// 192 in 16 pieces (32 us; small tiles 40).
struct TileCost {
  uint32_t step, tile, tile_z;     // a K step, a tile, a tile that updates z
  uint32_t tail;                   // the partials of a tail
  uint32_t piece, piece_t, even;   // those of K pieces: in all, per tile; in all without a tail
};

template <int EPI>
HILO_DEV uint32_t plan_cost(uint32_t T, uint32_t nk, TileCost c) {
  constexpr uint32_t P = kGemmWorkgroups;
  const uint32_t rounds = (T + P - 1) / P, t = EPI == EPI_RESID ? c.tile_z : c.tile;
  if (runs_whole(T, nk)) return rounds * (nk * c.step + t) + (EPI == EPI_RESID ? 300 : 700);
  const uint32_t steps = T * nk / P * c.step;
  if (T >= P) return steps + rounds * t + c.tail;
  return steps + ((T & (T - 1)) == 0 ? c.even : c.piece + c.piece_t * T);
}

enum Tile { TILE_192, TILE_256, TILE_SMALL };

// The tile and its row tiles.  Nothing here divides by a value that is not a constant: every launch
// waits for this, about 2 us when it formed the three plans instead.
template <int EPI>
HILO_DEV Tile choose_tile(const GemmProblem &p, int &rows) {
  constexpr uint32_t P = kGemmWorkgroups;
  int r64 = 0, r192 = 0, r256 = 0;
  for (int s = 0; s < p.B; ++s) {
    const int img = cu_at(p.cu, s + 1) - p.L - cu_at(p.cu, s);
    r64 += (img + 63) / 64 + (p.L + 63) / 64;
    r192 += (img + 191) / 192 + (p.L + 191) / 192;
    r256 += (img + 255) / 256 + (p.L + 255) / 256;
  }
  const uint32_t nk = p.K / 64, tiles = uint32_t(r64) * (p.N / 32);
  uint32_t best = plan_cost<EPI>(r192 * ((p.N + 191) / 192), nk, TileCost{91, 400, 1400, 2000, 2700, 20, 2500});
  rows = r192;
  Tile t = TILE_192;
  const uint32_t c256 = plan_cost<EPI>(r256 * ((p.N + 255) / 256), nk, TileCost{146, 700, 3300, 3600, 4500, 35, 4500});
  if (c256 < best) {
    best = c256;
    rows = r256;
    t = TILE_256;
  }
  // a turn takes 2 tiles a workgroup; with one the K steps run twice as fast
  const uint32_t turns = (tiles + 2 * P - 1) / (2 * P);
  if (turns * ((nk + 3) / 4 * (tiles <= P ? 140 : 265) + 300) < best) {
    rows = r64;
    t = TILE_SMALL;
  }
  return t;
}

template <int BM, int BN, int EPI, int ROLE>
__global__ __launch_bounds__(512, 2) void k_gemm8_fp8(GemmProblem p) {
  __shared__ __attribute__((aligned(1024))) uint8_t lds[g8::Geo<BM, BN, true>::LDS];
  const int pid = xcd_remap(blockIdx.x, kGemmWorkgroups);
  gemm8_run<BM, BN, EPI, true>(p, sk_plan(p, row_tiles_total(p, BM), BN, 128), pid, lds);
}

template <int EPI, int ROLE>
__global__ __launch_bounds__(512, 2) void k_gemm8(GemmProblem p) {
  constexpr int L0 = g8::Geo<192, 192>::LDS, L1 = g8::Geo<256, 256>::LDS;
  __shared__ __attribute__((aligned(1024))) uint8_t lds[L0 > L1 ? L0 : L1];
  const int pid = xcd_remap(blockIdx.x, kGemmWorkgroups);
  int rows;
  switch (choose_tile<EPI>(p, rows)) {
    case TILE_SMALL: gemm_small_run<EPI>(p, rows, pid, lds); break;
    case TILE_256: gemm8_run<256, 256, EPI>(p, sk_plan(p, rows, 256), pid, lds); break;
    default: gemm8_run<192, 192, EPI>(p, sk_plan(p, rows, 192), pid, lds);
  }
}

// Finishes every tile left in partials.  A work item is one fragment row of one main-kernel wave
// of one tile, taken by one wave of the fixup: it adds the tile's partials (pieces in K order,
// stream-K contributors in workgroup order) and runs the epilogue on the row.  Contributions are
// loaded in batches of four (one memory round trip per batch instead of per contributor) and
// added in the fixed order, so the result does not depend on the batching.  A tile of the 8-wave kernels has 48
// items, so that 22 cut tiles already keep 4 waves a workgroup busy twice over: with 8, FP8 MLP down (K 9216) at
// 200 rows takes 37.8 us against 41.9, at 1800 rows 68.9 against 75.2, and a launch that finds nothing costs the
// same.
constexpr int kFixThreads = 512;
constexpr int kFixBatch = 4;

template <int BM, int BN, int WM, int WN, bool CONTIG, int EPI, bool F8>
HILO_DEV void gemm_fix(const GemmProblem &p, const SkPlan &q) {
  constexpr int P = kGemmWorkgroups;
  if (q.s == 1 && q.I == 0) return;  // every tile was finished by the main kernel
  using T = SkTile<BM, BN, WM, WN, CONTIG>;
  constexpr int TM = T::TM, TN = T::TN, NW = T::NW, FW = kFixThreads / 64;
  const int nfix = q.s > 1 ? q.T : q.U - q.dp;
  const int lane = threadIdx.x & 63;
  const int items = nfix * NW * TM;
  for (int x = blockIdx.x * FW + (threadIdx.x >> 6); x < items; x += gridDim.x * FW) {
    const int f = x / (NW * TM), rem = x - f * (NW * TM), wid = rem / TM, i = rem - wid * TM;
    const int t = q.s > 1 ? f : q.dp + f;
    f32x4 acc[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const float *b[kFixBatch];
    int nb = 0;
    auto flush = [&]() {
      f32x4 v[kFixBatch][TN];
#pragma unroll
      for (int c = 0; c < kFixBatch; ++c)
        if (c < nb) {
#pragma unroll
          for (int j = 0; j < TN; ++j) v[c][j] = *reinterpret_cast<const f32x4 *>(b[c] + T::part_index(wid, i, j, lane));
        }
#pragma unroll
      for (int c = 0; c < kFixBatch; ++c)
        if (c < nb) {
#pragma unroll
          for (int j = 0; j < TN; ++j) acc[j] += v[c][j];
        }
      nb = 0;
    };
    auto push = [&](const float *slot) {
#pragma unroll
      for (int c = 0; c < kFixBatch; ++c)
        if (c == nb) b[c] = slot;
      if (++nb == kFixBatch) flush();
    };
    bool done_whole = false;
    for (int pc = 0; pc < q.s; ++pc) {
      const int u = pc * q.T + t;
      if (u < q.dp) {
        push(p.part + size_t(u) * T::kPartFloats);
        continue;
      }
      const int v = u - q.dp;
      const long long a0 = (long long)v * q.len;
      const int w0 = sk_owner(q.I, q.Pk, a0), w1 = sk_owner(q.I, q.Pk, a0 + q.len - 1);
      if (q.s == 1 && w0 == w1) {  // one workgroup held the whole tile and finished it
        done_whole = true;
        break;
      }
      // contributors in workgroup order.  Range starts floor(I w / Pk) advance by additions (no
      // 64-bit division per contributor); a range's first unit is v exactly when it starts at or
      // after unit v's first iteration.
      const int Pk = q.Pk;
      const long long qI = q.I / Pk, rI = q.I - qI * Pk;
      long long qb = q.I * w0 / Pk, rb = q.I * w0 - qb * Pk;
      for (int w = w0; w <= w1; ++w) {
        long long qn = qb + qI, rn = rb + rI;
        if (rn >= Pk) {
          ++qn;
          rn -= Pk;
        }
        if (qb < qn) push(p.part + (size_t(P) + size_t(w) * 2 + (qb >= a0 ? 0 : 1)) * T::kPartFloats);
        qb = qn;
        rb = rn;
      }
    }
    if (done_whole) continue;
    flush();
    int rt, tn;
    tile_coords(q, t, rt, tn);
    const TileRows tr = decode_row_tile(p, BM, rt);
    if constexpr (F8 && EPI == EPI_BIAS && BN == 256) {
      if (p.qk8 != nullptr && tn * BN < 2 * p.D) {
        T::epilogue_row_qk8(p, tr, tn * BN, wid, i, lane, acc);
        continue;
      }
    }
    T::template epilogue_row<EPI, F8>(p, tr, tn * BN, wid, i, lane, acc);
  }
}

template <int BM, int BN, int EPI, int ROLE>
__global__ __launch_bounds__(kFixThreads) void k_gemm8_fp8_fix(GemmProblem p) {
  using G = g8::Geo<BM, BN, true>;
  gemm_fix<BM, BN, G::WM, G::WN, !G::B32, EPI, true>(p, sk_plan(p, row_tiles_total(p, BM), BN, 128));
}

template <int EPI, int ROLE>
__global__ __launch_bounds__(kFixThreads) void k_gemm8_fix(GemmProblem p) {
  int rows;
  const Tile t = choose_tile<EPI>(p, rows);
  if (t == TILE_256) gemm_fix<256, 256, 2, 4, true, EPI, false>(p, sk_plan(p, rows, 256));
  else if (t == TILE_192) gemm_fix<192, 192, 2, 4, true, EPI, false>(p, sk_plan(p, rows, 192));
}

// ------------------------------------------------------------------------------- fp32 path

// v_mfma_f32_16x16x4_f32 on fragments read straight from global memory: lane (r, g) = (l % 16, l / 16)
// takes 16 bytes of row r at K offset 4 g of every 16, and MFMA j of the four multiplies element j of
// both operands (any order of K will do as long as both agree), so no LDS staging and no barrier
// stands between the loads and the matrix core.  A workgroup's tile is 32 x 32 and its 4 waves take a
// quarter of K each (their sums meet in LDS): the float32 problems are small, and what bounds them is
// the serial chain of one wave -- K / 16 steps of 16 MFMAs -- and too few waves, not bandwidth.
// 551 rows (32 x 32 grid, D 256, MLP 1024), against the LDS-tiled scalar FMA kernel on 64 x 64 tiles
// before: QKV 29.7 -> 8.5 us, output 30 -> 6, MLP up 33 -> 11, MLP down 110 -> 12.5.
template <int EPI>
__global__ __launch_bounds__(256) void k_gemm_f32(GemmProblem p) {
  constexpr int BM = 32, BN = 32, CH = 4;  // CH: 16-deep K steps loaded ahead
  __shared__ f32x4 part[4][4][64];
  // tiles of the rows that are there, so that the XCDs share them evenly; the grid is sized for the
  // longest sequences
  const int tilesN = p.N / BN, tiles = row_tiles_total(p, BM) * tilesN;
  for (int b = blockIdx.x; b < tiles; b += gridDim.x) {
    const int tile = xcd_remap(b, tiles), tn = tile % tilesN;
    const TileRows tr = decode_row_tile(p, BM, tile / tilesN);
    const int n0 = tn * BN;  // N % 64 == 0: the tile's columns all exist
    const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lr = lane & 15, lg = lane >> 4;
    const float *A[2], *W[2];
  #pragma unroll
    for (int i = 0; i < 2; ++i) {
      A[i] = reinterpret_cast<const float *>(p.A) + size_t(tr.row0 + min(16 * i + lr, tr.nrows - 1)) * p.lda + 4 * lg;
      W[i] = reinterpret_cast<const float *>(tr.sigma ? p.W[1] : p.W[0]) + size_t(n0 + 16 * i + lr) * p.K + 4 * lg;
    }
    const int steps = p.K / 16, s0 = steps * wid / 4, s1 = steps * (wid + 1) / 4;  // K % 64 == 0: never empty
    f32x4 acc[2][2];
  #pragma unroll
    for (int i = 0; i < 2; ++i)
  #pragma unroll
      for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto load = [&](int s, f32x4 (&a)[CH][2], f32x4 (&w)[CH][2]) __attribute__((always_inline)) {
  #pragma unroll
      for (int c = 0; c < CH; ++c) {
        const int k = 16 * min(s + c, s1 - 1);  // past the wave's range: re-read its last step
  #pragma unroll
        for (int i = 0; i < 2; ++i) {
          a[c][i] = *reinterpret_cast<const f32x4 *>(A[i] + k);
          w[c][i] = *reinterpret_cast<const f32x4 *>(W[i] + k);
        }
      }
    };
    auto mul = [&](int s, const f32x4 (&a)[CH][2], const f32x4 (&w)[CH][2]) __attribute__((always_inline)) {
  #pragma unroll
      for (int c = 0; c < CH; ++c)
        if (s + c < s1) {
  #pragma unroll
          for (int e = 0; e < 4; ++e)
  #pragma unroll
            for (int i = 0; i < 2; ++i)
  #pragma unroll
              for (int j = 0; j < 2; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[c][j][e], a[c][i][e], acc[i][j], 0, 0, 0);
        }
    };
    f32x4 xa[CH][2], xw[CH][2], ya[CH][2], yw[CH][2];
    load(s0, xa, xw);
  #pragma unroll 1
    for (int s = s0; s < s1; s += 2 * CH) {
      if (s + CH < s1) load(s + CH, ya, yw);
      mul(s, xa, xw);
      if (s + CH >= s1) break;
      if (s + 2 * CH < s1) load(s + 2 * CH, xa, xw);
      mul(s + CH, ya, yw);
    }
  #pragma unroll
    for (int i = 0; i < 2; ++i)
  #pragma unroll
      for (int j = 0; j < 2; ++j) part[wid][2 * i + j][lane] = acc[i][j];
    __syncthreads();
    // wave w finishes subtile w: rows 16 (w / 2) + lr, columns 16 (w % 2) + 4 lg .. + 3
    const f32x4 v = (part[0][wid][lane] + part[1][wid][lane]) + (part[2][wid][lane] + part[3][wid][lane]);
    const int rl = 16 * (wid >> 1) + lr;
    const float out[4] = {v[0], v[1], v[2], v[3]};
    if (rl < tr.nrows) epilogue4<EPI, false>(p, tr, tr.row0 + rl, n0 + 16 * (wid & 1) + 4 * lg, out);
    __syncthreads();  // the next tile's waves write the same LDS
  }
}

// ------------------------------------------------------------------------------- dispatch

// FP8: one persistent workgroup per CU, BM x BN tiles.
template <int BM, int BN, int ROLE>
static hipError_t run_fp8(const GemmProblem &p, hipStream_t st) {
  static_assert(size_t(BM) * BN * 3 * kGemmWorkgroups * sizeof(float) <= kSkPartBytes, "partial area too small");
  constexpr int P = kGemmWorkgroups;
  hipLaunchKernelGGL((k_gemm8_fp8<BM, BN, role_epilogue(ROLE), ROLE>), dim3(P), dim3(512), 0, st, p);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const long long tiles_max = (long long)p.B * ((p.max_img_rows + BM - 1) / BM + (p.L + BM - 1) / BM) *
                              ((p.N + BN - 1) / BN);
  if (tiles_max < P && p.K / 128 <= kNoSplitSteps) return hipSuccess;
  // P workgroups stride over the fixup's items: few enough that a launch with nothing to finish
  // (the device's row counts led to whole tiles) costs little
  hipLaunchKernelGGL((k_gemm8_fp8_fix<BM, BN, role_epilogue(ROLE), ROLE>), dim3(P), dim3(kFixThreads), 0, st, p);
  return hipGetLastError();
}

// bf16: one persistent workgroup per CU, the tile chosen on the device.
template <int ROLE>
static hipError_t run_bf16(const GemmProblem &p, hipStream_t st) {
  constexpr int P = kGemmWorkgroups;
  hipLaunchKernelGGL((k_gemm8<role_epilogue(ROLE), ROLE>), dim3(P), dim3(512), 0, st, p);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // no tile is ever cut when even 192 x 192 tiles are fewer than workgroups and K is short
  const long long tiles_max = (long long)p.B * ((p.max_img_rows + 191) / 192 + (p.L + 191) / 192) * ((p.N + 191) / 192);
  if (tiles_max < P && p.K / 64 <= kNoSplitSteps) return hipSuccess;
  hipLaunchKernelGGL((k_gemm8_fix<role_epilogue(ROLE), ROLE>), dim3(P), dim3(kFixThreads), 0, st, p);
  return hipGetLastError();
}

template <int EPI>
static hipError_t run_f32(const GemmProblem &p, hipStream_t st) {
  const long long nblk = (long long)p.B * ((p.max_img_rows + 31) / 32 + (p.L + 31) / 32) * (p.N / 32);
  if (nblk <= 0) return hipSuccess;
  // the grid is bounded (its threads must stay below 2^32); larger problems loop
  hipLaunchKernelGGL((k_gemm_f32<EPI>), dim3(unsigned(nblk < (1 << 20) ? nblk : (1 << 20))), dim3(256), 0, st, p);
  return hipGetLastError();
}

hipError_t launch_gemm(bool bf16, int role, const GemmProblem &p, hipStream_t st) {
  if (!bf16) {
    switch (role_epilogue(role)) {
      case EPI_BIAS: return run_f32<EPI_BIAS>(p, st);
      case EPI_GELU: return run_f32<EPI_GELU>(p, st);
      default: return run_f32<EPI_RESID>(p, st);
    }
  }
  switch (role) {
    case GEMM_QKV: return run_bf16<GEMM_QKV>(p, st);
    case GEMM_O: return run_bf16<GEMM_O>(p, st);
    case GEMM_FC1: return run_bf16<GEMM_FC1>(p, st);
    default: return run_bf16<GEMM_FC2>(p, st);
  }
}

hipError_t launch_gemm_fp8(int role, const GemmProblem &p, hipStream_t st) {
  switch (role) {
    // the FP8 QKV projection always writes FP8 q / k: 256-column tiles (whole heads per wave)
    case GEMM_QKV: return p.qk8 ? run_fp8<256, 256, GEMM_QKV>(p, st) : hipErrorInvalidValue;
    case GEMM_O: return run_fp8<192, 192, GEMM_O>(p, st);
    case GEMM_FC1: return run_fp8<192, 192, GEMM_FC1>(p, st);
    default: return run_fp8<192, 192, GEMM_FC2>(p, st);
  }
}

}  // namespace hilo
