// Dense projections of the prefill: C[M, N] = A[M, K] . W[N, K]^T with fused
// epilogues (rotary embedding on q/k, SwiGLU, GELU, residual add).
//
// bf16 / fp16 path (gfx950 MFMA): 256 x 256 output tile per 256-thread
// workgroup (one per CU), K stepped by 64 through two LDS stages (2 x 64 KB)
// filled by 16-byte direct-to-LDS loads.  Four waves, one per SIMD, in a
// 2 x 2 grid each own a 128 x 128 sub-tile = 4 x 4 blocks of
// v_mfma_f32_32x32x16 (256 accumulator registers per lane).  The next
// stage's loads are spread over the MFMAs of the first three quarters of the
// current one (a burst of them stalls the wave's MFMA issue), and each wave's loads
// go to 4 KB-contiguous LDS runs so one M0 value serves four of them through
// the instruction's immediate offset.  The next tile's first stage is
// fetched while the epilogue of the current one runs.
//
// M (tokens in the chunk) is read from device memory; the grid is persistent
// (one workgroup per CU) and walks the tiles, so an empty chunk costs one
// launch and no work.  Where M leaves 256 x 256 tiles too few for the chip the
// same launch takes 128 x 128 or 64 x 64 ones, also for the rows that would fill the
// last round of large tiles in part (tile_plan).
//
// fp32 path: 32 x 64 tiles on the fp32 matrix instructions with the same row
// mapping, used for fp32 models.
#include "aiq_internal.h"
#include "dev_util.h"

#include <type_traits>

namespace aiq {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));

static int g_cus[64];

static int num_cus() {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  if (g_cus[dev] == 0) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
    g_cus[dev] = n;
  }
  return g_cus[dev];
}


__device__ __forceinline__ float gelu_erf(float x) { return 0.5f * x * (1.0f + erff(x * 0.70710678118654752f)); }

// Row of the q or k weight that produces GEMM column c of that section.
// For hd = 128 the two 64-column halves of a head are reordered so that one
// wave's 64 columns hold 32 complete rotary pairs (i, i + 64).
__device__ __forceinline__ int qk_row(int c, int hd) {
  if (hd != 128) return c;   // 64-dim heads: natural order
  const int head = c >> 7, cc = c & 127;
  const int hh = cc >> 6, jj = cc & 63;
  const int dim = jj < 32 ? hh * 32 + jj : 64 + hh * 32 + (jj - 32);
  return head * 128 + dim;
}

template <int EPI, typename T>
__device__ __forceinline__ const T* b_row(const GemmArgs& a, int n) {
  if (EPI == EPI_QKV_ROPE) {
    // the bf16 kernel applies the rotary pairs in registers and needs the
    // reordered rows; the fp32 kernel keeps the natural order
    constexpr bool reorder = sizeof(T) == 2;
    if (n < a.n_q) return static_cast<const T*>(a.B0) + static_cast<int64_t>(reorder ? qk_row(n, a.hd) : n) * a.K;
    n -= a.n_q;
    if (n < a.n_kv) return static_cast<const T*>(a.B1) + static_cast<int64_t>(reorder ? qk_row(n, a.hd) : n) * a.K;
    n -= a.n_kv;
    return static_cast<const T*>(a.B2) + static_cast<int64_t>(n) * a.K;
  } else if (EPI == EPI_SWIGLU) {
    // interleave 32-row groups: gate rows 32b.., up rows 32b.., ... so each
    // 64-column wave slice holds 32 gate columns and the 32 matching up columns
    const int b32 = n >> 5, r = n & 31;
    const int row = (b32 >> 1) * 32 + r;
    return static_cast<const T*>((b32 & 1) ? a.B1 : a.B0) + static_cast<int64_t>(row) * a.K;
  } else {
    return static_cast<const T*>(a.B0) + static_cast<int64_t>(n) * a.K;
  }
}

// ======================================================================= 16-bit MFMA
// The MFMA path runs on bf16 or fp16 operands (H = fp16); both forms of
// v_mfma_f32_32x32x16 have the same rate.
template <bool H> struct Op16;
template <> struct Op16<false> {
  typedef bf16x8 V;
  static __device__ __forceinline__ f32x16_t mma(V a, V b, f32x16_t c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ uint16_t cvt(float f) { return f2bf(f); }
  static __device__ __forceinline__ float widen(uint16_t u) { return __uint_as_float(static_cast<uint32_t>(u) << 16); }
};
template <> struct Op16<true> {
  typedef half8 V;
  static __device__ __forceinline__ f32x16_t mma(V a, V b, f32x16_t c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ uint16_t cvt(float f) { return f2h(f); }
  static __device__ __forceinline__ float widen(uint16_t u) { return h2f(u); }
};
constexpr int GM = 256, GN = 256, GK = 64, GT = 256;

typedef f32x16_t f32x16;

// Accumulator layout.  The MFMAs compute the transposed tile, weights as the
// first operand (v_mfma_f32_32x32x16: D[r][c] with r = 8g + 4*(lane/32) + e
// in register 4g + e, c = lane % 32): acc[i][j][4g + e] holds C[m][n] with
//   m = m0 + wm*128 + i*32 + lane%32,   n = n0 + wn*128 + j*32 + 8g + 4*(lane/32) + e,
// four consecutive columns of one row per (j, g).
//
// Epilogue: for each 32-row block i the wave writes its 32 x 128 fp32
// accumulators to its own 16 KB slice of the idle LDS stage, 16 bytes per
// (j, g) straight from the accumulator registers, then reads them back as
// pieces of 8 consecutive columns of one row, 16 consecutive lanes covering
// one row, so every global access of the epilogue is a contiguous run of
// 256 or 512 bytes per row.  The SwiGLU pair (columns c and c + 32 of a
// 64-column half: gate and up) and the rotary pair (lower and upper half of
// a head's dims, as the q/k weight rows are reordered) are pieces 4 apart.
//
// q, k and v (attention operands) are stored in fp16: 10 mantissa bits where
// bf16 has 7, at the same MFMA rate; their magnitudes are O(1) after RMSNorm.

// The residual epilogue's butterfly of DPP moves (dpp_f32) takes the same
// partners and adds in the same order as lane ^ 1, ^ 2, ^ 4 shuffles: after
// the first two steps the four lanes of a quad hold equal sums, so the
// mirrored quad is the ^ 4 partner's.

__device__ __forceinline__ float silu_fast(float g) {
  return g * __builtin_amdgcn_rcpf(1.0f + __expf(-g));
}

template <bool H>
__device__ __forceinline__ uint4 pack8(const float (&v)[8]) {
  uint4 p;
  p.x = Op16<H>::cvt(v[0]) | (static_cast<uint32_t>(Op16<H>::cvt(v[1])) << 16);
  p.y = Op16<H>::cvt(v[2]) | (static_cast<uint32_t>(Op16<H>::cvt(v[3])) << 16);
  p.z = Op16<H>::cvt(v[4]) | (static_cast<uint32_t>(Op16<H>::cvt(v[5])) << 16);
  p.w = Op16<H>::cvt(v[6]) | (static_cast<uint32_t>(Op16<H>::cvt(v[7])) << 16);
  return p;
}
__device__ __forceinline__ uint4 pack8h(const float (&v)[8]) {
  uint4 p;
  p.x = f2h(v[0]) | (static_cast<uint32_t>(f2h(v[1])) << 16);
  p.y = f2h(v[2]) | (static_cast<uint32_t>(f2h(v[3])) << 16);
  p.z = f2h(v[4]) | (static_cast<uint32_t>(f2h(v[5])) << 16);
  p.w = f2h(v[6]) | (static_cast<uint32_t>(f2h(v[7])) << 16);
  return p;
}

// The wave's epilogue slice: 32 rows x 128 fp32, 512-byte rows of 32
// 16-byte chunks; chunk c of row r sits at slot c ^ (r & 15), so 16
// consecutive rows writing one chunk, and one row read by 16 lanes, each
// cover all 64 banks.
__device__ __forceinline__ int eslot(int r, int c) { return r * 32 + (c ^ (r & 15)); }

// Makes this wave's LDS writes visible to its own later reads in other
// lanes (LDS completes one wave's operations in order; this keeps the
// compiler from moving them across).
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---- epilogues of one 8-column piece (columns c .. c + 7 of row m; `in`: m < M)
// x += acc in place; with a following norm also h = x * g and, per 64
// columns (eight neighbouring lanes, in a fixed butterfly order), the sum of
// x^2.  g0, g1: the norm's gains of the columns.
template <int EPI, bool H>
__device__ __forceinline__ void resid_piece(const GemmArgs& a, float4 x0, float4 x1, const float4& s0,
                                            const float4& s1, const float4& g0, const float4& g1, int64_t m, int c,
                                            bool in, int pc, bool norm, uint16_t* hout) {
  x0.x += s0.x; x0.y += s0.y; x0.z += s0.z; x0.w += s0.w;
  x1.x += s1.x; x1.y += s1.y; x1.z += s1.z; x1.w += s1.w;
  float ssq = 0.f;
  if (in) {
    float* xr = a.x + m * a.ldc + c;
    *reinterpret_cast<float4*>(xr) = x0;
    *reinterpret_cast<float4*>(xr + 4) = x1;
    if (norm) {
      const float hv[8] = {x0.x * g0.x, x0.y * g0.y, x0.z * g0.z, x0.w * g0.w,
                           x1.x * g1.x, x1.y * g1.y, x1.z * g1.z, x1.w * g1.w};
      *reinterpret_cast<uint4*>(hout + m * a.ldc + c) = pack8<H>(hv);
    }
    ssq = ((x0.x * x0.x + x0.y * x0.y) + (x0.z * x0.z + x0.w * x0.w)) +
          ((x1.x * x1.x + x1.y * x1.y) + (x1.z * x1.z + x1.w * x1.w));
  }
  if (norm) {
    ssq += dpp_f32<0xB1>(ssq);    // quad_perm [1,0,3,2]: lane ^ 1
    ssq += dpp_f32<0x4E>(ssq);    // quad_perm [2,3,0,1]: lane ^ 2
    ssq += dpp_f32<0x141>(ssq);   // row_half_mirror: the other quad of the eight, whose lanes agree
    if ((pc & 7) == 0 && in) a.ssp[m * a.n_part + (c >> 6)] = ssq;
  }
}

// Row maximum over each 64 columns: the lane's 8 columns in increasing order
// (a strictly greater value replaces), then eight lanes in a butterfly that
// keeps the lower column on ties.
__device__ __forceinline__ void argmax_piece(const GemmArgs& a, const float4& s0, const float4& s1, int64_t m,
                                             int col, bool in, int pc) {
  const float v8[8] = {s0.x, s0.y, s0.z, s0.w, s1.x, s1.y, s1.z, s1.w};
  float v = v8[0];
  int c = col;
#pragma unroll
  for (int e = 1; e < 8; ++e)
    if (v8[e] > v) {
      v = v8[e];
      c = col + e;
    }
#pragma unroll
  for (int o = 1; o < 8; o <<= 1) {
    const float ov = __shfl_xor(v, o);
    const int oc = __shfl_xor(c, o);
    if (ov > v || (ov == v && oc < c)) {
      v = ov;
      c = oc;
    }
  }
  if ((pc & 7) == 0 && in) static_cast<int2*>(a.C)[m * a.ldc + (col >> 6)] = make_int2(__float_as_int(v), c);
}

template <int EPI, bool H>
__device__ __forceinline__ void store_piece(const GemmArgs& a, const float4& s0, const float4& s1, int64_t m, int c) {
  if (EPI == EPI_STORE_F32) {
    float* cr = static_cast<float*>(a.C) + m * a.ldc + c;
    *reinterpret_cast<float4*>(cr) = s0;
    *reinterpret_cast<float4*>(cr + 4) = s1;
  } else {
    const float v8[8] = {s0.x, s0.y, s0.z, s0.w, s1.x, s1.y, s1.z, s1.w};
    *reinterpret_cast<uint4*>(static_cast<uint16_t*>(a.C) + m * a.ldc + c) = pack8<H>(v8);
  }
}

// SwiGLU and rotary pairs: pieces q and q + 4 of the 64-column half that
// starts at column nh (gate and up; lower and upper half dims), scaled by the
// row's RMSNorm scale rs.  rv: rotary frequencies of a head's lower dims.
template <int EPI, bool H>
__device__ __forceinline__ void pair_piece(const GemmArgs& a, const float4& l0, const float4& l1, const float4& u0,
                                           const float4& u1, float rs, int nh, int q, int64_t m, int32_t position,
                                           const float* rv) {
  const float lo[8] = {l0.x * rs, l0.y * rs, l0.z * rs, l0.w * rs, l1.x * rs, l1.y * rs, l1.z * rs, l1.w * rs};
  const float up[8] = {u0.x * rs, u0.y * rs, u0.z * rs, u0.w * rs, u1.x * rs, u1.y * rs, u1.z * rs, u1.w * rs};
  uint16_t* crow = static_cast<uint16_t*>(a.C) + m * a.ldc;
  if (EPI == EPI_SWIGLU) {
    float o[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = silu_fast(lo[e]) * up[e];
    *reinterpret_cast<uint4*>(crow + (nh >> 1) + 8 * q) = pack8<H>(o);
  } else if (nh >= a.n_q + a.n_kv) {   // v: natural order
    *reinterpret_cast<uint4*>(crow + nh + 8 * q) = pack8h(lo);
    *reinterpret_cast<uint4*>(crow + nh + 32 + 8 * q) = pack8h(up);
  } else {
    const int sbase = nh < a.n_q ? 0 : a.n_q;
    // 64- or 128-dim heads: column nh of a section is the head's own (hh 0) or second 64-column half
    const int hh = a.hd == 128 ? ((nh - sbase) >> 6) & 1 : 0, half = a.hd >> 1;
    const float pos = static_cast<float>(position);
    const float4 f0 = *reinterpret_cast<const float4*>(rv + hh * 32 + 8 * q);
    const float4 f1 = *reinterpret_cast<const float4*>(rv + hh * 32 + 8 * q + 4);
    const float fr[8] = {f0.x, f0.y, f0.z, f0.w, f1.x, f1.y, f1.z, f1.w};
    float ol[8], ou[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      // angle pos * theta^(-2i/hd), in revolutions (hardware sin/cos take revolutions)
      const float rev = pos * fr[e];
      const float frac = rev - floorf(rev);
      const float cs = __builtin_amdgcn_cosf(frac), sn = __builtin_amdgcn_sinf(frac);
      ol[e] = lo[e] * cs - up[e] * sn;   // lower half dim
      ou[e] = up[e] * cs + lo[e] * sn;   // upper half dim
    }
    uint16_t* dst = crow + nh - hh * 32 + 8 * q;
    *reinterpret_cast<uint4*>(dst) = pack8h(ol);
    *reinterpret_cast<uint4*>(dst + half) = pack8h(ou);
  }
}

// `rl` holds the tile's row scales (QKV, SwiGLU) or the following norm's gain
// for the tile's columns (residual), `pl` the tile's positions and `rv` the
// rotary frequencies of a head's lower-half dims (revolutions per position),
// all in LDS; `slice` is the wave's 16 KB of idle LDS.  `prefetch` issues the
// next tile's first loads (after the residual epilogue's first loads of x,
// so that those do not queue behind it; first for the others).
template <int EPI, bool H, typename Prefetch>
__device__ __forceinline__ void epilogue_bf16(const GemmArgs& a, f32x16 (&acc)[4][4], int64_t m0, int n0,
                                              int64_t M, int wm, int wn, int lane, float4* slice, const float* rl,
                                              const int32_t* pl, const float* rv, int64_t tok0, Prefetch prefetch) {
  const int l32 = lane & 31, hi = lane >> 5;
  const int nw = n0 + wn * 128;   // first GEMM column of the wave's sub-tile
  const int pc = lane & 15;       // piece (8 columns) of a row this lane reads back
  const int pr = lane >> 4;       // its row inside each group of 4 rows
  constexpr bool RESID = EPI == EPI_RESID || EPI == EPI_RESID_EMB;
  if (!RESID) prefetch();
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    // fp32 accumulators of rows 32i .. 32i + 31 to LDS
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        slice[eslot(l32, 8 * j + 2 * g + hi)] =
            make_float4(acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]);
    wave_lds_sync();
    const int row0 = wm * 128 + i * 32;   // tile row of slice row 0
    if (RESID) {
      // x += acc in place; with a following norm also h = x * g and, per row,
      // the sum of x^2 over each 64-column half (pieces 8h .. 8h + 7, eight
      // neighbouring lanes, added in a fixed butterfly order).  All eight
      // rows' residuals of this lane are read before any is used.
      const bool norm = a.gnext != nullptr;
      uint16_t* hout = static_cast<uint16_t*>(a.hout);
      const int col = nw + 8 * pc;
      float4 xv[8][2];
#pragma unroll
      for (int rr = 0; rr < 8; ++rr) {
        int64_t m = m0 + row0 + 4 * rr + pr;
        if (m > M - 1) m = M - 1;   // in bounds; the value is not used
        if (EPI == EPI_RESID_EMB) {
          // the residual before this projection is the token's embedding row
          // widened from 16 bits, which is exactly what x would hold
          int32_t tok = a.x_tok[tok0 + m];
          if (tok < 0 || tok >= a.vocab) tok = 0;
          const uint4 e = *reinterpret_cast<const uint4*>(static_cast<const uint16_t*>(a.x_emb) +
                                                          static_cast<int64_t>(tok) * a.ldc + col);
          xv[rr][0] = make_float4(Op16<H>::widen(static_cast<uint16_t>(e.x & 0xFFFFu)),
                                  Op16<H>::widen(static_cast<uint16_t>(e.x >> 16)),
                                  Op16<H>::widen(static_cast<uint16_t>(e.y & 0xFFFFu)),
                                  Op16<H>::widen(static_cast<uint16_t>(e.y >> 16)));
          xv[rr][1] = make_float4(Op16<H>::widen(static_cast<uint16_t>(e.z & 0xFFFFu)),
                                  Op16<H>::widen(static_cast<uint16_t>(e.z >> 16)),
                                  Op16<H>::widen(static_cast<uint16_t>(e.w & 0xFFFFu)),
                                  Op16<H>::widen(static_cast<uint16_t>(e.w >> 16)));
        } else {
          const float* xr = a.x + m * a.ldc + col;
          xv[rr][0] = *reinterpret_cast<const float4*>(xr);
          xv[rr][1] = *reinterpret_cast<const float4*>(xr + 4);
        }
      }
      if (i == 0) prefetch();
      float4 g0 = make_float4(0.f, 0.f, 0.f, 0.f), g1 = g0;
      if (norm) {
        g0 = *reinterpret_cast<const float4*>(rl + (col - n0));
        g1 = *reinterpret_cast<const float4*>(rl + (col - n0) + 4);
      }
#pragma unroll
      for (int rr = 0; rr < 8; ++rr) {
        const int r = 4 * rr + pr;
        const int64_t m = m0 + row0 + r;
        float4 x0 = xv[rr][0], x1 = xv[rr][1];
        const float4 s0 = slice[eslot(r, 2 * pc)], s1 = slice[eslot(r, 2 * pc + 1)];
        resid_piece<EPI, H>(a, x0, x1, s0, s1, g0, g1, m, col, m < M, pc, norm, hout);
      }
    } else if (EPI != EPI_SWIGLU && EPI != EPI_QKV_ROPE) {
#pragma unroll
      for (int rr = 0; rr < 8; ++rr) {
        const int r = 4 * rr + pr;
        const int64_t m = m0 + row0 + r;
        const float4 s0 = slice[eslot(r, 2 * pc)], s1 = slice[eslot(r, 2 * pc + 1)];
        if (EPI == EPI_ARGMAX)
          argmax_piece(a, s0, s1, m, nw + 8 * pc, m < M, pc);
        else if (m < M)
          store_piece<EPI, H>(a, s0, s1, m, nw + 8 * pc);
      }
    } else {
      // pieces q (0..3) and q + 4 of one 64-column half h; lane piece pc ->
      // (h, q) = (pc / 8, pc % 4) on rows of parity pc / 4 % 2: 32 rows x 2
      // halves x 4 pairs = 256 pair-pieces, 4 per lane
      const int h = pc >> 3, q = pc & 3, rp = (pc >> 2) & 1;
#pragma unroll
      for (int rr = 0; rr < 4; ++rr) {
        const int r = 8 * rr + 2 * pr + rp;
        const int tr = row0 + r;
        const float rs = a.rs ? rl[tr] : 1.f;   // RMSNorm row scale
        const float4 l0 = slice[eslot(r, 16 * h + 2 * q)], l1 = slice[eslot(r, 16 * h + 2 * q + 1)];
        const float4 u0 = slice[eslot(r, 16 * h + 2 * q + 8)], u1 = slice[eslot(r, 16 * h + 2 * q + 9)];
        if (m0 + tr < M) pair_piece<EPI, H>(a, l0, l1, u0, u1, rs, nw + 64 * h, q, m0 + tr, pl[tr], rv);
      }
    }
    wave_lds_sync();   // the slice's reads are done before the next block's writes
  }
}

typedef __attribute__((address_space(3))) void* lds_ptr_t;

// LDS stage: [256 rows][64 bf16], 128-byte rows of eight 16-byte chunks.  The
// chunk index is XORed with bits 1..3 of the row: 16 consecutive rows then
// cover all 64 banks once (row parity already picks the bank half).
__device__ __forceinline__ int swz(int row, int chunk) { return chunk ^ ((row >> 1) & 7); }

// Fragments of one 16-deep sub-step s of the wave's 128 x 128 sub-tile.
template <bool H>
__device__ __forceinline__ void load_frags(const uint16_t* As, const uint16_t* Bs, int s, int wm, int wn, int lane,
                                           typename Op16<H>::V (&af)[4], typename Op16<H>::V (&bw)[4]) {
  typedef typename Op16<H>::V V;
  const int r32 = lane & 31;
  const int sw = swz(r32, 2 * s + (lane >> 5)) << 3;   // same for every 32-row block
#pragma unroll
  for (int i = 0; i < 4; ++i) af[i] = *reinterpret_cast<const V*>(As + (wm * 128 + i * 32 + r32) * GK + sw);
#pragma unroll
  for (int j = 0; j < 4; ++j) bw[j] = *reinterpret_cast<const V*>(Bs + (wn * 128 + j * 32 + r32) * GK + sw);
}

// 16-byte direct-to-LDS load whose immediate offset, (i % 4) KB, is added to
// both the global and the LDS address (the global pointer carries -(i % 4) KB).
__device__ __forceinline__ void load_lds_imm(const void* g, lds_ptr_t l, int i) {
  switch (i & 3) {
    case 0: __builtin_amdgcn_global_load_lds(g, l, 16, 0, 0); break;
    case 1: __builtin_amdgcn_global_load_lds(g, l, 16, 1024, 0); break;
    case 2: __builtin_amdgcn_global_load_lds(g, l, 16, 2048, 0); break;
    default: __builtin_amdgcn_global_load_lds(g, l, 16, 3072, 0); break;
  }
}

// Global -> LDS copy of one stage: wave w fills rows 64w .. 64w + 63 of A and
// of W (eight 1 KB pieces of 8 rows each); in a piece's instruction lane l
// fetches the global chunk that belongs at row 8c + l/8, slot l%8.  The
// source pointers advance by one k-step.
__device__ __forceinline__ void dma_stage(uint16_t* sA, uint16_t* sB, const uint16_t* (&ga)[8],
                                          const uint16_t* (&gb)[8], int w) {
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int c = 8 * w + (i & 4);
    load_lds_imm(static_cast<const void*>(ga[i]), (lds_ptr_t)(sA + c * 512), i);
    load_lds_imm(static_cast<const void*>(gb[i]), (lds_ptr_t)(sB + c * 512), i);
    ga[i] += GK;
    gb[i] += GK;
  }
}

// One 64-deep k-step of the wave's sub-tile from one LDS stage (4 sub-steps of
// 16 MFMAs).  Fragments of the next sub-step are read while the MFMAs of the
// current one run, and the next stage's 16 loads (8 pieces of A, then 8 of
// W) go out during the first three sub-steps, 5, 5 and 6 of them, each after
// an MFMA.  Issued over two sub-steps, the loads back up in the memory
// pipeline and stall MFMA issue on large problems (4 % slower at 2M rows);
// issued over all four, the last ones are still in flight at the stage's
// closing barrier.  The source pointers point at the k-block after the one
// being consumed; `dma` is false in the tile's last stage, when they are one
// past the row's end.  The loads then re-read the row's last k-block into the
// idle stage and the pointers stay, so every stage runs the same
// straight-line schedule (a branch around the loads splits the stage into
// blocks that the scheduler cannot interleave: 1-2 % slower).
template <bool H>
__device__ __forceinline__ void mma_stage(const uint16_t* As, const uint16_t* Bs, f32x16 (&acc)[4][4], int wm,
                                          int wn, int lane, uint16_t* nA, uint16_t* nB, const uint16_t* (&ga)[8],
                                          const uint16_t* (&gb)[8], int w, bool dma) {
  typename Op16<H>::V af[2][4], bw[2][4];
  load_frags<H>(As, Bs, 0, wm, wn, lane, af[0], bw[0]);
  __builtin_amdgcn_sched_barrier(0);   // the first sub-step's reads are not interleaved with its own MFMAs
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const int cur = s & 1;
    if (s < 3) load_frags<H>(As, Bs, s + 1, wm, wn, lane, af[cur ^ 1], bw[cur ^ 1]);
    const int l0 = (16 * s) / 3, l1 = s < 3 ? (16 * (s + 1)) / 3 : l0;   // this sub-step's loads [l0, l1)
    const int back = dma ? 0 : -GK, adv = dma ? GK : 0;
#pragma unroll
    for (int l = l0; l < l1; ++l) {
      const int i = l & 7, c = 8 * w + (i & 4);
      if (l < 8) {
        load_lds_imm(static_cast<const void*>(ga[i] + back), (lds_ptr_t)(nA + c * 512), i);
        ga[i] += adv;
      } else {
        load_lds_imm(static_cast<const void*>(gb[i] + back), (lds_ptr_t)(nB + c * 512), i);
        gb[i] += adv;
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        acc[i][j] = Op16<H>::mma(bw[cur][j], af[cur][i], acc[i][j]);
    // the first 8 MFMAs each followed by one fragment read and (while any
    // are left) one load, then the other 8
    for (int q = 0; q < 8; ++q) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                  // MFMA
      if (s < 3) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);       // DS read
      if (q < l1 - l0) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0); // VMEM read
    }
    __builtin_amdgcn_sched_group_barrier(0x008, 8, 0);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// Source pointers of a tile's first k-step (see dma_stage), each carrying
// -(i % 4) KB for the loads' immediate offset.
template <int EPI>
__device__ __forceinline__ void tile_sources(const GemmArgs& a, const uint16_t* A, int64_t M, int64_t m0, int n0,
                                             int w, int lane, const uint16_t* (&ga)[8], const uint16_t* (&gb)[8]) {
  const int lr = lane >> 3;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int row = (8 * w + i) * 8 + lr;
    const int lc = swz(row, lane & 7);   // logical chunk stored in this lane's slot
    // rows past M are never stored; they read the tile row above (256-row
    // tiles run only with M >= GM), not all one row: that many requests for one
    // cache line serialise in the L2 (3.5x the time of a whole launch)
    int64_t mr = m0 + row;
    if (mr > M - 1) mr -= GM;
    ga[i] = A + mr * a.lda + lc * 8 - (i & 3) * 512;
    gb[i] = b_row<EPI, uint16_t>(a, n0 + row) + lc * 8 - (i & 3) * 512;
  }
}

// ----------------------------------------------------------------- small tiles
// Few rows leave most of the chip idle with 256 x 256 tiles (M = 120, N = 512:
// two tiles).  The same kernel then walks BM x BN = 64 x 64 or 128 x 128
// tiles, four waves in a 2 x 2 grid, K in 32 KB stages (SLABS slabs of 64)
// through a ring of four: three stages of loads in flight per workgroup
// instead of one, since here the memory latency per stage is what counts.
// Every output is still one accumulator over K in order with the same MFMA,
// so a row's bits do not depend on which tile shape ran it.
//
// Rows of A past M are not read at all (buffer loads, out of range).
constexpr int ST_BYTES = 32768;   // one stage: SLABS x (A [BM][64] | W [BN][64])

template <int N>
__device__ __forceinline__ void wait_vm_barrier() {
  // this wave's loads but the last N have landed and its LDS reads are done;
  // then every wave's
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

// Direct-to-LDS loads, 16 bytes per lane to 1 KB at LDS byte `dst` (uniform).
// In asm: the compiler would wait for every load in flight before each read
// of a stage (it cannot tell the ring's stages apart across iterations);
// wait_vm_barrier does the waiting.  No register is written.
__device__ __forceinline__ uint32_t lds_offset(const void* p) {
  return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_ptr_t)p));
}
__device__ __forceinline__ void dma_global(const void* src, uint32_t dst) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(dst), "v"(src)
               : "memory", "m0");
}
__device__ __forceinline__ void dma_buffer(int __attribute__((ext_vector_type(4))) rsrc, int voff, int soff, uint32_t dst) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(dst), "v"(voff),
               "s"(rsrc), "s"(soff)
               : "memory", "m0");
}

// 16-byte chunk c of row r of the finished tile in LDS.
template <int BN>
__device__ __forceinline__ int tslot(int r, int c) { return r * (BN / 4) + (c ^ (r & 15)); }

template <int EPI, bool H, int BM, int BN, int SLABS>
__device__ __forceinline__ void gemm_tiles(const GemmArgs& a, int64_t mb, int64_t M, uint16_t* st0, uint16_t* st1, uint16_t* st2,
                                           uint16_t* st3, float* rbuf, int32_t* pbuf, const float* rvbuf) {
  static_assert(SLABS * (BM + BN) * GK * 2 == ST_BYTES, "stage size");
  typedef typename Op16<H>::V V;
  constexpr int WI = BM / 64, WJ = BN / 64;   // 32 x 32 blocks per wave
  constexpr int LD = ST_BYTES / 4096;         // 1 KB loads per wave and stage
  constexpr bool RESID = EPI == EPI_RESID || EPI == EPI_RESID_EMB;
  constexpr bool PAIR = EPI == EPI_SWIGLU || EPI == EPI_QKV_ROPE;
  constexpr int PPR = BN / 8;                 // pieces per row
  constexpr int NP = BM * PPR / GT;           // pieces per thread
  const int t = threadIdx.x, lane = t & 63, w = t >> 6, wm = w >> 1, wn = w & 1;
  const int l32 = lane & 31, hi = lane >> 5, lr = lane >> 3;
  static_assert(BM == BN, "each wave copies as many pieces of A as of W");
  const int tiles_n = a.N / BN;
  const int tiles_m = static_cast<int>((M - mb + BM - 1) / BM);   // rows mb .. M - 1
  const int tiles = tiles_m * tiles_n;
  const int ns = a.K / (GK * SLABS);
  // XCD x takes a contiguous eighth of the tiles in column-major order: equal
  // shares for every M, and one XCD's workgroups share weight columns
  const int xcd = blockIdx.x & 7, per_xcd = gridDim.x >> 3;
  const int lo = static_cast<int>(static_cast<int64_t>(tiles) * xcd / 8);
  const int end = static_cast<int>(static_cast<int64_t>(tiles) * (xcd + 1) / 8);
  uint16_t* const stv[4] = {st0, st1, st2, st3};

  for (int tile = lo + static_cast<int>(blockIdx.x >> 3); tile < end; tile += per_xcd) {
    const int col = tile / tiles_m;
    const int64_t m0 = mb + static_cast<int64_t>(tile - col * tiles_m) * BM;
    const int n0 = col * BN;
    const int rows = M - m0 < BM ? static_cast<int>(M - m0) : BM;
    __syncthreads();   // the previous tile's epilogue is done with the stages, rbuf and pbuf
    // the residual of this thread's pieces, in flight under the k loop
    float4 xv[RESID ? NP : 1][2];
    if (RESID) {
      const int64_t tok0 = EPI == EPI_RESID_EMB ? a.x_tok_desc[D_TOK_BEGIN] : 0;
#pragma unroll
      for (int u = 0; u < NP; ++u) {
        const int p = t + u * GT, r = p / PPR, c = n0 + 8 * (p % PPR);
        const int64_t m = m0 + (r < rows ? r : 0);
        if (EPI == EPI_RESID_EMB) {
          int32_t tok = a.x_tok[tok0 + m];
          if (tok < 0 || tok >= a.vocab) tok = 0;
          const uint4 e = *reinterpret_cast<const uint4*>(static_cast<const uint16_t*>(a.x_emb) +
                                                          static_cast<int64_t>(tok) * a.ldc + c);
          xv[u][0] = make_float4(Op16<H>::widen(static_cast<uint16_t>(e.x & 0xFFFFu)),
                                 Op16<H>::widen(static_cast<uint16_t>(e.x >> 16)),
                                 Op16<H>::widen(static_cast<uint16_t>(e.y & 0xFFFFu)),
                                 Op16<H>::widen(static_cast<uint16_t>(e.y >> 16)));
          xv[u][1] = make_float4(Op16<H>::widen(static_cast<uint16_t>(e.z & 0xFFFFu)),
                                 Op16<H>::widen(static_cast<uint16_t>(e.z >> 16)),
                                 Op16<H>::widen(static_cast<uint16_t>(e.w & 0xFFFFu)),
                                 Op16<H>::widen(static_cast<uint16_t>(e.w >> 16)));
        } else {
          const float* xr = a.x + m * a.ldc + c;
          xv[u][0] = *reinterpret_cast<const float4*>(xr);
          xv[u][1] = *reinterpret_cast<const float4*>(xr + 4);
        }
      }
    }
    if (PAIR && t < BM) {
      if (a.ssp_in)
        rbuf[t] = row_scale(a.ssp_in + (m0 + (t < rows ? t : 0)) * (a.K / 64), a.K / 64, a.K, a.eps);
      else if (a.rs)
        rbuf[t] = a.rs[m0 + t];   // padded by 256 rows
    }
    if (RESID && a.gnext && t < BN) rbuf[t] = a.gnext[n0 + t];
    if (EPI == EPI_QKV_ROPE && t < BM) pbuf[t] = a.pos[m0 + t];

    // sources: of each stage this wave copies LD / 2 pieces (8 rows x 64 k) of
    // A and as many of W
    typedef int v4i __attribute__((ext_vector_type(4)));
    const uint64_t abase = reinterpret_cast<uint64_t>(static_cast<const uint16_t*>(a.A) + m0 * a.lda);
    v4i ra;   // buffer over the tile's rows below M
    ra[0] = __builtin_amdgcn_readfirstlane(static_cast<int>(abase));
    ra[1] = __builtin_amdgcn_readfirstlane(static_cast<int>(abase >> 32));
    ra[2] = __builtin_amdgcn_readfirstlane(static_cast<int>(rows * a.lda * 2));
    ra[3] = 0x00020000;
    const uint16_t* gb[LD / 2];
    int ao[LD / 2];
    uint32_t so[LD / 2];   // the A piece's place in a stage; W's is BM * GK elements further
#pragma unroll
    for (int i = 0; i < LD / 2; ++i) {
      const int p = (LD / 2) * w + i, slab = p / (BM / 8), row = (p % (BM / 8)) * 8 + lr;
      const int kk = slab * GK + swz(row, lane & 7) * 8;
      ao[i] = static_cast<int>((row * a.lda + kk) * 2);
      gb[i] = b_row<EPI, uint16_t>(a, n0 + row) + kk;
      so[i] = static_cast<uint32_t>(slab * (BM + BN) * GK + (p % (BM / 8)) * 8 * GK) * 2;
    }
    auto load_stage = [&](int s, const uint16_t* st) {
      const uint32_t base = lds_offset(st);
#pragma unroll
      for (int i = 0; i < LD / 2; ++i) {
        const uint32_t d = __builtin_amdgcn_readfirstlane(base + so[i]);
        dma_buffer(ra, ao[i], s * (GK * SLABS * 2), d);
        dma_global(gb[i] + s * (GK * SLABS), d + BM * GK * 2);
      }
    };
    f32x16 acc[WI][WJ];
#pragma unroll
    for (int i = 0; i < WI; ++i)
#pragma unroll
      for (int j = 0; j < WJ; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
    auto compute = [&](const uint16_t* st) {
      // all fragments of the stage are requested before its first MFMA, which
      // then wait only for their own
      V af[SLABS * 4][WI], bw[SLABS * 4][WJ];
#pragma unroll
      for (int s = 0; s < SLABS * 4; ++s) {
        const uint16_t* As = st + (s >> 2) * (BM + BN) * GK;
        const uint16_t* Bs = As + BM * GK;
        const int sw = swz(l32, 2 * (s & 3) + hi) << 3;
#pragma unroll
        for (int i = 0; i < WI; ++i)
          af[s][i] = *reinterpret_cast<const V*>(As + (wm * (BM / 2) + i * 32 + l32) * GK + sw);
#pragma unroll
        for (int j = 0; j < WJ; ++j)
          bw[s][j] = *reinterpret_cast<const V*>(Bs + (wn * (BN / 2) + j * 32 + l32) * GK + sw);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int s = 0; s < SLABS * 4; ++s)
#pragma unroll
        for (int i = 0; i < WI; ++i)
#pragma unroll
          for (int j = 0; j < WJ; ++j) acc[i][j] = Op16<H>::mma(bw[s][j], af[s][i], acc[i][j]);
    };
#pragma unroll
    for (int s = 0; s < 3; ++s)
      if (s < ns) load_stage(s, stv[s]);
    auto step = [&](int s, uint16_t* cur, uint16_t* nxt) {
      // stage s has landed everywhere and every wave is done with stage s - 1,
      // whose buffer takes stage s + 3
      if (s + 2 < ns)
        wait_vm_barrier<2 * LD>();
      else if (s + 1 < ns)
        wait_vm_barrier<LD>();
      else
        wait_vm_barrier<0>();
      if (s + 3 < ns) load_stage(s + 3, nxt);
      compute(cur);
    };
    for (int s = 0; s < ns; s += 4) {
      step(s, st0, st3);
      if (s + 1 < ns) step(s + 1, st1, st0);
      if (s + 2 < ns) step(s + 2, st2, st1);
      if (s + 3 < ns) step(s + 3, st3, st2);
    }
    __syncthreads();   // every wave is done with the stages: they take the tile in fp32
    float4* const tl = reinterpret_cast<float4*>(st0);
    float4* const th = reinterpret_cast<float4*>(st1);   // rows 64.. of a 128-row tile
#pragma unroll
    for (int i = 0; i < WI; ++i)
#pragma unroll
      for (int j = 0; j < WJ; ++j)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int r = wm * (BM / 2) + i * 32 + l32;
          (r < 64 ? tl : th)[tslot<BN>(r & 63, wn * (BN / 8) + 8 * j + 2 * g + hi)] =
              make_float4(acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]);
        }
    __syncthreads();
    auto rd = [&](int r, int c) { return (r < 64 ? tl : th)[tslot<BN>(r & 63, c)]; };
    if (!PAIR) {
#pragma unroll
      for (int u = 0; u < NP; ++u) {
        const int p = t + u * GT, r = p / PPR, pc = p % PPR;
        const int64_t m = m0 + r;
        const int c = n0 + 8 * pc;
        const bool in = r < rows;
        const float4 s0 = rd(r, 2 * pc), s1 = rd(r, 2 * pc + 1);
        if (RESID)
          resid_piece<EPI, H>(a, xv[u][0], xv[u][1], s0, s1, *reinterpret_cast<const float4*>(rbuf + 8 * pc),
                              *reinterpret_cast<const float4*>(rbuf + 8 * pc + 4), m, c, in, pc, a.gnext != nullptr,
                              static_cast<uint16_t*>(a.hout));
        else if (EPI == EPI_ARGMAX)
          argmax_piece(a, s0, s1, m, c, in, pc);
        else if (in)
          store_piece<EPI, H>(a, s0, s1, m, c);
      }
    } else {
      constexpr int QPR = BN / 16;   // pair-pieces per row: 4 per 64-column half
#pragma unroll
      for (int u = 0; u < BM * QPR / GT; ++u) {
        const int p = t + u * GT, r = p / QPR, h = (p % QPR) >> 2, q = p & 3;
        const float rs = a.rs || a.ssp_in ? rbuf[r] : 1.f;
        const float4 l0 = rd(r, 16 * h + 2 * q), l1 = rd(r, 16 * h + 2 * q + 1);
        const float4 u0 = rd(r, 16 * h + 2 * q + 8), u1 = rd(r, 16 * h + 2 * q + 9);
        if (r < rows) pair_piece<EPI, H>(a, l0, l1, u0, u1, rs, n0 + 64 * h, q, m0 + r, pbuf[r], rvbuf);
      }
    }
  }
}

// Which tiles a launch of M rows takes: 256 x 256 ones for the rows before the
// returned one, 128 x 128 or 64 x 64 (`t64`) for the others, by the rounds over
// the grid.  Costs in microseconds of one round, per 64-deep k-step and for
// start plus epilogue, fitted to single rounds at K = 512 .. 8192 with cold
// weights: 64 x 64 tiles 0.21 / 2.2 (10 us at K = 2048, 30 at 8192), 128 x 128
// 0.53 / 4.5 (21, 69), 256 x 256 1.44 / 11 (60, 196; the maxima epilogue
// takes 15).  The 256-row tiles' rounds count by XCD, whose rows they are
// dealt to in turn.  They also need a whole tile of rows (the sources of rows past M) and row
// scales, not sums (`large`).
// Measured at K = 3072, N = 3072: M = 120 17 us against 92 with the large
// tiles only, M = 800 37 against 91, M = 1920 70 against 91, M = 3300 112
// against 93.  Where the last round of large tiles would be partly empty, the rows
// past the last whole one go to small tiles: N = 2048, K = 8192, M = 18,200 (2.25 rounds)
// 608 us against 670, N = 512, K = 2048, M = 66,000 195 against 236.
template <int EPI>
__device__ __forceinline__ int64_t tile_plan(int64_t M, int N, int K, int wgs, bool large, bool& t64) {
  auto rounds = [](int64_t tiles, int slots) {
    return static_cast<float>(static_cast<uint32_t>(tiles + slots - 1) / static_cast<uint32_t>(slots));
  };
  const float k = static_cast<float>(K / GK);
  const int tn64 = N / 64, tn128 = N / 128, tn = N / GN, per = wgs >> 3;
  auto c64 = [&](int64_t m) { return rounds((m + 63) / 64 * tn64, wgs) * (0.21f * k + 2.2f); };
  auto c128 = [&](int64_t m) { return rounds((m + 127) / 128 * tn128, wgs) * (0.53f * k + 4.5f); };
  const float e256 = 1.44f * k + (EPI == EPI_ARGMAX ? 15.f : 11.f);
  int64_t m1 = 0;
  if (large && M >= GM) {
    m1 = M;
    float best = rounds(((M + GM - 1) / GM + 7) / 8 * tn, per) * e256;
    if (M < 65536) {   // all rows small only pays where there are few rounds
      const float all = fminf(c64(M), c128(M));
      if (all < best) {
        best = all;
        m1 = 0;
      }
    }
    const int64_t rx = M / (8 * GM);   // whole tile rows per XCD
#pragma unroll 1
    for (int64_t r = rx; r > 0 && r > rx - 8; --r) {
      const int64_t rest = M - r * (8 * GM);
      const float c = rounds(r * tn, per) * e256 + (rest ? fminf(c64(rest), c128(rest)) : 0.f);
      if (c < 0.97f * best) {
        best = c;
        m1 = r * (8 * GM);
      }
    }
  }
  t64 = c64(M - m1) <= c128(M - m1);
  return m1;
}

template <int EPI, bool H>
__global__ __launch_bounds__(GT, 1) void k_gemm_bf16(GemmArgs a) {
  // two stages in distinct arrays: the compiler can then tell the in-flight
  // loads into one stage from the reads of the other and only waits at the
  // barrier that ends the stage
  __shared__ __attribute__((aligned(16))) uint16_t sA0[GM * GK];
  __shared__ __attribute__((aligned(16))) uint16_t sB0[GN * GK];
  __shared__ __attribute__((aligned(16))) uint16_t sA1[GM * GK];
  __shared__ __attribute__((aligned(16))) uint16_t sB1[GN * GK];
  __shared__ __attribute__((aligned(16))) float rbuf[GM];     // the tile's RMSNorm row scales
  __shared__ __attribute__((aligned(16))) int32_t pbuf[GM];   // the tile's token positions (QKV)
  __shared__ __attribute__((aligned(16))) float rvbuf[64];    // rotary frequencies of the lower-half dims (QKV)
  const int64_t M = *a.m_ptr;
  if (M <= 0) return;
  const int64_t tok0 = EPI == EPI_RESID_EMB ? a.x_tok_desc[D_TOK_BEGIN] : 0;   // the rows' first packed token
  if (EPI == EPI_QKV_ROPE && static_cast<int>(threadIdx.x) < (a.hd >> 1))
    rvbuf[threadIdx.x] = a.rope_rev[threadIdx.x];   // visible after the first barrier
  bool t64;
  const int64_t M1 = tile_plan<EPI>(M, a.N, a.K, gridDim.x, !a.ssp_in, t64);   // rows of 256-row tiles
  const int tiles_n = a.N / GN;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6, wm = w >> 1, wn = w & 1;
  const int nk = a.K / GK;   // even (the launcher checks K % 128)
  const uint16_t* A = static_cast<const uint16_t*>(a.A);

  // XCD-aware order: workgroups are dispatched round-robin over the 8 XCDs,
  // so workgroup b runs on XCD b % 8.  XCD x owns the M-tile rows
  // tm = x, x + 8, x + 16, ...; inside an XCD the tiles go in groups of
  // group_m of its rows, column by column, so the 32 workgroups resident on
  // one XCD share a few activation row-panels and a few weight column-panels
  // in that XCD's L2 instead of streaming 32 distinct panels.  Groups of 2
  // rows (gate/up 1-1.8 %, O 1-3.6 %, down 0.6-1.8 % faster than 4), 4 for
  // the q|k|v projection (2 is 2-3 % slower there).
  constexpr int group_m = EPI == EPI_QKV_ROPE ? 4 : 2;
  const int tiles_m = static_cast<int>((M1 + GM - 1) / GM);   // < 2^31 (M < 2^39)
  const int xcd = blockIdx.x & 7;
  const int per_xcd = gridDim.x >> 3;   // grid is a multiple of 8
  const int rows_x = tiles_m > xcd ? (tiles_m - xcd + 7) / 8 : 0;
  const int count_x = rows_x * tiles_n;
  const unsigned per_group = static_cast<unsigned>(group_m * tiles_n);
  auto tile_mn = [&](int q, int64_t& m0, int& n0) {
    const unsigned grp = static_cast<unsigned>(q) / per_group, within = static_cast<unsigned>(q) - grp * per_group;
    const int left = rows_x - static_cast<int>(grp) * group_m;
    const unsigned rows_here = left < group_m ? static_cast<unsigned>(left) : static_cast<unsigned>(group_m);   // 1 .. 4
    unsigned col, r;
    switch (rows_here) {   // within / rows_here without a division
      case 4: col = within >> 2; r = within & 3; break;
      case 2: col = within >> 1; r = within & 1; break;
      case 1: col = within; r = 0; break;
      default: col = within / 3; r = within - col * 3; break;
    }
    const int lr = static_cast<int>(grp) * group_m + static_cast<int>(r);
    m0 = static_cast<int64_t>(lr * 8 + xcd) * GM;
    n0 = static_cast<int>(col) * GN;
  };
  int q = blockIdx.x >> 3;
  const uint16_t* ga[8];
  const uint16_t* gb[8];
  int64_t m0 = 0;
  int n0 = 0;
  if (q < count_x) {
    tile_mn(q, m0, n0);
    tile_sources<EPI>(a, A, M, m0, n0, w, lane, ga, gb);
    dma_stage(sA0, sB0, ga, gb, w);
  }
  for (; q < count_x; q += per_xcd) {
    f32x16 acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
    __syncthreads();   // stage 0 of this tile has landed; the last epilogue is done with rbuf / pbuf
    // the tile's row scales and positions go to LDS now, so that the epilogue
    // reads no global memory behind the next tile's prefetch
    if (w == 0 && (EPI == EPI_QKV_ROPE || EPI == EPI_SWIGLU) && a.rs)
      __builtin_amdgcn_global_load_lds(static_cast<const void*>(a.rs + m0 + lane * 4), (lds_ptr_t)(rbuf + lane * 4),
                                       16, 0, 0);
    if (w == 0 && (EPI == EPI_RESID || EPI == EPI_RESID_EMB) && a.gnext)   // the following norm's gain for the tile's columns
      __builtin_amdgcn_global_load_lds(static_cast<const void*>(a.gnext + n0 + lane * 4),
                                       (lds_ptr_t)(rbuf + lane * 4), 16, 0, 0);
    if (w == 1 && EPI == EPI_QKV_ROPE)
      __builtin_amdgcn_global_load_lds(static_cast<const void*>(a.pos + m0 + lane * 4), (lds_ptr_t)(pbuf + lane * 4),
                                       16, 0, 0);
    // nk is even: stages alternate 0, 1 and the loop has no odd tail (a
    // conditional second stage makes the compiler move the accumulators
    // between register files every iteration)
    for (int kt = 0; kt < nk; kt += 2) {
      mma_stage<H>(sA0, sB0, acc, wm, wn, lane, sA1, sB1, ga, gb, w, true);
      __syncthreads();
      mma_stage<H>(sA1, sB1, acc, wm, wn, lane, sA0, sB0, ga, gb, w, kt + 2 < nk);
      __syncthreads();
    }
    // stage 0 is free: the next tile's first k-step loads under the epilogue
    const bool more = q + per_xcd < count_x;
    int64_t m1 = 0;
    int n1 = 0;
    if (more) tile_mn(q + per_xcd, m1, n1);
    auto prefetch = [&]() {
      if (more) {
        tile_sources<EPI>(a, A, M, m1, n1, w, lane, ga, gb);
        dma_stage(sA0, sB0, ga, gb, w);
      }
    };
    // each wave stages its accumulators in its own 16 KB of stage 1, which is
    // idle until the next tile's first barrier
    float4* slice = reinterpret_cast<float4*>((w < 2 ? sA1 : sB1) + (w & 1) * 8192);
    epilogue_bf16<EPI, H>(a, acc, m0, n0, M, wm, wn, lane, slice, rbuf, pbuf, rvbuf, tok0, prefetch);
    m0 = m1;
    n0 = n1;
  }
  // the last tile's re-read of its last k-block lands before the workgroup
  // gives up its LDS
  __builtin_amdgcn_s_waitcnt(0);
  if (M1 >= M) return;
  if (t64)
    gemm_tiles<EPI, H, 64, 64, 2>(a, M1, M, sA0, sB0, sA1, sB1, rbuf, pbuf, rvbuf);
  else
    gemm_tiles<EPI, H, 128, 128, 1>(a, M1, M, sA0, sB0, sA1, sB1, rbuf, pbuf, rvbuf);
}

hipError_t launch_gemm_bf16(int epi, const GemmArgs& a, hipStream_t s) {
  if (a.K <= 0 || a.K % (2 * GK) || a.N % GN) return hipErrorInvalidValue;   // whole pairs of k-steps, whole tiles
  if (a.ssp_in && a.K % 256) return hipErrorInvalidValue;                    // sums read four at a time
  // one workgroup per CU, rounded to whole XCD groups; fewer for small problems
  const int64_t tiles = ((a.m_ub + 63) / 64) * (a.N / 64);   // the smallest tiles
  int64_t g = num_cus();
  if (tiles < g) g = tiles;
  g = (g + 7) / 8 * 8;
  const dim3 grid(static_cast<unsigned>(g)), block(GT);
#define AIQ_LAUNCH_GEMM(E)                                                         \
  do {                                                                             \
    if (a.f16)                                                                     \
      hipLaunchKernelGGL((k_gemm_bf16<E, true>), grid, block, 0, s, a);            \
    else                                                                           \
      hipLaunchKernelGGL((k_gemm_bf16<E, false>), grid, block, 0, s, a);           \
  } while (0)
  switch (epi) {
    case EPI_STORE_F32: AIQ_LAUNCH_GEMM(EPI_STORE_F32); break;
    case EPI_ARGMAX:
      if (a.ldc != a.N / 64) return hipErrorInvalidValue;
      AIQ_LAUNCH_GEMM(EPI_ARGMAX);
      break;
    case EPI_STORE_ACT: AIQ_LAUNCH_GEMM(EPI_STORE_ACT); break;
    case EPI_SWIGLU: AIQ_LAUNCH_GEMM(EPI_SWIGLU); break;
    case EPI_QKV_ROPE: AIQ_LAUNCH_GEMM(EPI_QKV_ROPE); break;
    case EPI_RESID:
    case EPI_RESID_EMB:
      if (a.ldc != a.N || a.N % 64 || (a.gnext && (!a.hout || !a.ssp || a.n_part != a.N / 64)))
        return hipErrorInvalidValue;
      if (epi == EPI_RESID_EMB) {
        if (!a.x_emb || !a.x_tok || !a.x_tok_desc || a.vocab <= 0) return hipErrorInvalidValue;
        AIQ_LAUNCH_GEMM(EPI_RESID_EMB);
      } else {
        AIQ_LAUNCH_GEMM(EPI_RESID);
      }
      break;
    default: return hipErrorInvalidValue;
  }
#undef AIQ_LAUNCH_GEMM
  return hipGetLastError();
}

// ======================================================================= fp32
// 32 x 64 tile per workgroup, four waves in a 2 x 2 grid of 16 x 32, on
// v_mfma_f32_16x16x4_f32 (fp32 products and sums).  fp32 models are small
// (N = 128 .. 512, a few thousand rows): a launch is bound by latency, so the
// tile is small (338 workgroups at M = 5,392, N = 128), K goes in steps of 64
// through two LDS stages with the next step's global loads in flight, and one
// barrier per step.  M = 5,392: K = 512 58 us with the former 64 x 64 FMA tile
// (K in steps of 16, nothing in flight) and 15.5 us with this.
constexpr int FM = 32, FN = 64, FK = 64, FP = FK + 4, FT = 256;   // FP: row pitch in LDS, conflict-free

template <int EPI>
__global__ __launch_bounds__(FT) void k_gemm_f32(GemmArgs a) {
  __shared__ __attribute__((aligned(16))) float S[2][(FM + FN) * FP];
  const int64_t M = *a.m_ptr;
  if (M <= 0) return;
  const int tiles_n = a.N / FN;
  const int64_t n_tiles = ((M + FM - 1) / FM) * tiles_n;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6, wm = w >> 1, wn = w & 1;
  const int l16 = lane & 15, g = lane >> 4;
  const float* A = static_cast<const float*>(a.A);
  const int lrow = t >> 4, lk = (t & 15) * 4;   // this thread's rows lrow, lrow + 16, ... of a step, 4 floats each
  for (int64_t tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
    const int64_t m0 = (tile / tiles_n) * FM;
    const int n0 = static_cast<int>(tile % tiles_n) * FN;
    const float* src[6];
    bool ok[6];
#pragma unroll
    for (int u = 0; u < 6; ++u) {   // 2 x 16 rows of A, 4 x 16 of W
      const int row = lrow + 16 * (u < 2 ? u : u - 2);
      ok[u] = u >= 2 || m0 + row < M;
      src[u] = u < 2 ? A + (ok[u] ? m0 + row : 0) * a.lda + lk : b_row<EPI, float>(a, n0 + row) + lk;
    }
    float4 v[6];
    auto fetch = [&](int k0) {
#pragma unroll
      for (int u = 0; u < 6; ++u)
        v[u] = ok[u] ? *reinterpret_cast<const float4*>(src[u] + k0) : make_float4(0.f, 0.f, 0.f, 0.f);
    };
    f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
    fetch(0);
    int buf = 0;
    for (int k0 = 0; k0 < a.K; k0 += FK, buf ^= 1) {
      // buffer `buf` was last read before the barrier of the step before
      float* st = S[buf];
#pragma unroll
      for (int u = 0; u < 6; ++u) *reinterpret_cast<float4*>(st + (lrow + 16 * u) * FP + lk) = v[u];
      __syncthreads();
      if (k0 + FK < a.K) fetch(k0 + FK);
      const float* ar = st + (wm * 16 + l16) * FP + 4 * g;
      const float* br = st + (FM + wn * 32 + l16) * FP + 4 * g;
      // lane group g holds columns 16 s + 4 g .. + 3: product e of a 16-column
      // slice sums columns e, 4 + e, 8 + e, 12 + e
#pragma unroll
      for (int s = 0; s < FK / 16; ++s) {
        const f32x4 av = *reinterpret_cast<const f32x4*>(ar + 16 * s);
        const f32x4 b0 = *reinterpret_cast<const f32x4*>(br + 16 * s);
        const f32x4 b1 = *reinterpret_cast<const f32x4*>(br + 16 * FP + 16 * s);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(b0[e], av[e], acc[0], 0, 0, 0);
          acc[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(b1[e], av[e], acc[1], 0, 0, 0);
        }
      }
    }
    __syncthreads();   // both buffers free for the next tile
    // lane (l16, g): row l16 of the wave, columns 16 j + 4 g .. + 3
    const int64_t m = m0 + wm * 16 + l16;
    if (m < M) {
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        f32x4 o = acc[j];
        if (EPI == EPI_GELU) {
#pragma unroll
          for (int e = 0; e < 4; ++e) o[e] = gelu_erf(o[e]);
        }   // others: plain fp32 store (QKV columns in natural order; rotary applied afterwards)
        *reinterpret_cast<f32x4*>(static_cast<float*>(a.C) + m * a.ldc + n0 + wn * 32 + 16 * j + 4 * g) = o;
      }
    }
  }
}

hipError_t launch_gemm_f32(int epi, const GemmArgs& a, hipStream_t s) {
  if (a.K <= 0 || a.K % FK || a.N % FN) return hipErrorInvalidValue;   // whole k-steps, whole tiles
  const int64_t tiles = ((a.m_ub + FM - 1) / FM) * (a.N / FN);
  int64_t g = static_cast<int64_t>(num_cus()) * 4;
  if (tiles < g) g = tiles;
  if (g < 1) g = 1;
  const dim3 grid(static_cast<unsigned>(g)), block(FT);
  switch (epi) {
    case EPI_STORE_F32:
    case EPI_STORE_ACT: hipLaunchKernelGGL(k_gemm_f32<EPI_STORE_F32>, grid, block, 0, s, a); break;
    case EPI_QKV_ROPE: hipLaunchKernelGGL(k_gemm_f32<EPI_QKV_ROPE>, grid, block, 0, s, a); break;
    case EPI_GELU: hipLaunchKernelGGL(k_gemm_f32<EPI_GELU>, grid, block, 0, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// Rotary embedding in place on the q and k columns of an fp32 QKV buffer.
__global__ void k_rope_f32(const int64_t* desc, float* qkv, int64_t ld, int32_t n_q, int32_t n_kv, int32_t hd,
                           const int32_t* pos, const float* cos_t, const float* sin_t) {
  const int64_t nt = desc[D_NTOK];
  const int half = hd >> 1;
  const int heads = (n_q + n_kv) / hd;
  const int64_t total = nt * heads * half;
  for (int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; j < total; j += (int64_t)gridDim.x * blockDim.x) {
    const int i = static_cast<int>(j % half);
    const int64_t th = j / half;
    const int h = static_cast<int>(th % heads);
    const int64_t t = th / heads;
    float* base = qkv + t * ld + static_cast<int64_t>(h) * hd;   // q heads then k heads are contiguous
    const int64_t ti = static_cast<int64_t>(pos[t]) * half + i;
    const float c = cos_t[ti], s = sin_t[ti];
    const float x1 = base[i], x2 = base[i + half];
    base[i] = x1 * c - x2 * s;
    base[i + half] = x2 * c + x1 * s;
  }
}

hipError_t launch_rope_f32(const int64_t* desc, float* qkv, int64_t ld, int32_t n_q, int32_t n_kv,
                           int32_t hd, const int32_t* pos, const float* cos_t, const float* sin_t,
                           int64_t t_cap, hipStream_t s) {
  int64_t g = (t_cap * ((n_q + n_kv) / hd) * (hd / 2) + 255) / 256;
  if (g > 4096) g = 4096;
  if (g < 1) g = 1;
  hipLaunchKernelGGL(k_rope_f32, dim3(static_cast<unsigned>(g)), dim3(256), 0, s, desc, qkv, ld, n_q, n_kv, hd,
                     pos, cos_t, sin_t);
  return hipGetLastError();
}

}  // namespace aiq
