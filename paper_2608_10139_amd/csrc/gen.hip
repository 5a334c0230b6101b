// AI_TRANSFORM: greedy generation after the prefill (Table 1 maps it to a
// causal-LM forward with generative decoding, output masked with a pad id;
// Section 4, Q3 and Q5), and the LIKE match over the generated tokens.
//
// A generation step runs one row per sequence of the chunk through the same
// projections as the prefill (M = number of sequences), a decode attention
// kernel over the sequence's kept keys and values, and the full-vocabulary
// head as a GEMM whose epilogue keeps only each row's maximum per 64 columns,
// followed by a row argmax over those.  Keys and values
// of the prompt stay where the prefill put them (the chunk's per-layer q|k|v
// rows, plus the shared prefix's rows); those of generated tokens go to a
// per-layer cache [sequence][step][2 d_kv].  Everything runs on the launch
// stream; counts come from device memory.
#include "aiq_internal.h"
#include "dev_util.h"

#include <type_traits>

namespace aiq {

static int grid_for(int64_t n, int per_block, int cap) {
  int64_t g = (n + per_block - 1) / per_block;
  if (g < 1) g = 1;
  if (g > cap) g = cap;
  return static_cast<int>(g);
}

__device__ __forceinline__ float wave_sum_g(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// ------------------------------------------------------------------ descriptors
__global__ void k_gen_desc(const int64_t* cd, int64_t* gd, int64_t* cnt, int32_t nb) {
  const int64_t n = cd[D_NSEQ];
  if (threadIdx.x == 0) {
    gd[D_TOK_BEGIN] = 0;
    gd[D_NTOK] = n;
    gd[D_SEQ_BEGIN] = cd[D_SEQ_BEGIN];
    gd[D_NSEQ] = n;
  }
  for (int b = threadIdx.x; b < nb; b += blockDim.x) {
    const int64_t r = n - static_cast<int64_t>(b) * GEN_HEAD_ROWS;
    cnt[b] = r < 0 ? 0 : (r > GEN_HEAD_ROWS ? GEN_HEAD_ROWS : r);
  }
}

hipError_t launch_gen_desc(const int64_t* chunk_desc, int64_t* gen_desc, int64_t* cnt, int32_t n_blocks,
                           hipStream_t s) {
  hipLaunchKernelGGL(k_gen_desc, dim3(1), dim3(256), 0, s, chunk_desc, gen_desc, cnt, n_blocks);
  return hipGetLastError();
}

// ------------------------------------------------------------------ last positions of a chunk
// The label head needs only each sequence's last position, and in the last
// layer nothing after the q|k|v projection feeds any other position: that
// layer's attention (for the last query), O projection, norm and FFN run on
// one row per sequence, in blocks of R sequences.  Wave per sequence, 16-byte
// pieces of its rows.
__global__ __launch_bounds__(256) void k_last_rows(const int64_t* ld, const int64_t* cu, LastRows a) {
  const int64_t n = ld[D_NSEQ], sb = ld[D_SEQ_BEGIN], tb = ld[D_TOK_BEGIN];
  const int lane = threadIdx.x & 63;
  const int64_t wave = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6;
  const int64_t n_waves = ((int64_t)gridDim.x * blockDim.x) >> 6;
  const int d = a.d;
  for (int64_t i = wave; i < n; i += n_waves) {
    const int64_t c1 = cu[sb + i + 1];
    if (c1 == cu[sb + i]) continue;
    const int64_t r = c1 - 1 - tb;
    if (a.x) {
      const float4* src = reinterpret_cast<const float4*>(a.x + r * d);
      float4* dst = reinterpret_cast<float4*>(a.xl + i * d);
      for (int c = lane; c < d / 4; c += 64) dst[c] = src[c];
    }
    if (!a.hl) continue;
    const uint4* hs = reinterpret_cast<const uint4*>(static_cast<const uint16_t*>(a.h) + r * d);
    uint4* hd = reinterpret_cast<uint4*>(static_cast<uint16_t*>(a.hl) + i * d);
    for (int c = lane; c < d / 8; c += 64) hd[c] = hs[c];
    if (lane == 0) {
      a.rsl[i] = a.ssp ? row_scale(a.ssp + r * (d / 64), d / 64, d, a.eps) : a.rs[r];
      a.posl[i] = a.pos[r];
    }
  }
}

hipError_t launch_last_rows(const int64_t* ldesc, const int64_t* cu, const LastRows& a, int64_t R, hipStream_t s) {
  if (a.d % 8 || (a.hl && (!a.h || (!a.rs && !a.ssp) || (a.ssp && a.d % 256)))) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_last_rows, dim3(grid_for(R, 4, 8192)), dim3(256), 0, s, ldesc, cu, a);
  return hipGetLastError();
}

// ------------------------------------------------------------------ decode attention
// Workgroup per (sequence, K/V head): the REP = n_heads / n_kv query heads of
// the group against every kept key of the sequence (prompt, earlier generated
// tokens, this token).  A key row of HD fp16 values is read by LPK = HD / 8
// lanes, 16 bytes each, so one wave load covers 64 / LPK whole rows; keys go
// in blocks of 4 such loads, block b to share b mod 4, a share per wave (no second block in flight:
// its registers cost more in waves per SIMD, 3 for 5, than it hides).  Every lane group keeps its own
// running maximum and sum over the keys it reads, so a block needs no exchange
// between lanes but its dot products over the LPK lanes of a row (DPP moves);
// groups, then shares, merge at the end.  Bound: HBM for many sequences (each
// kept key and value row once), the chain of blocks for few.  One wave per
// item with the maximum and the sum of every block reduced over the wave
// through the LDS crossbar took 32 us per step for 256 sequences of 170 keys
// (8 heads of 64) and 98 us for 8 sequences of up to 585 (groups of 3, heads of
// 128); this takes 23 and 21 us.  The split depends on the keys alone, so a sequence's
// bits do not depend on the batch.  The workgroup also stores this step's key and
// value into the generated cache.
__device__ __forceinline__ float dpp_add(float v, int lanes) {
  v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0xB1, 0xF, 0xF, false));    // lane ^ 1
  v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x4E, 0xF, 0xF, false));    // lane ^ 2
  v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x141, 0xF, 0xF, false));   // the other quad of 8
  if (lanes == 16)
    v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x140, 0xF, 0xF, false));   // the other 8 of 16
  return v;
}

// v combined over the wave's lane groups of LPK (8 or 16) lanes, in every lane:
// the halves of 16-lane rows (row_ror:8), then v_permlane16_swap (rows paired)
// and v_permlane32_swap (halves of the wave); no LDS.
template <int LPK, typename F>
__device__ __forceinline__ float across_groups(float v, F f) {
  if (LPK == 8) v = f(v, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x128, 0xF, 0xF, false)));
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = f(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return f(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// Items from which on waves take them alone (groups of up to 3; wider ones keep a wave busy
// with registers): where they fill the chip several times over, and earlier where the longest
// prompt is short, since a long one is then a wave's serial chain.  A workgroup per item against
// waves alone, 8 K/V heads of 64: 2,000 sequences of 16 to 100 tokens 41 and 19 us, of 16 to
// 500 70 and 59, 1,000 22 and 13, 31 and 32, 500 13 and 10, 18 and 26, 250 7.3 and 8.0; 20,000 of
// two tokens 312 and 106.  Groups of 3, heads of 128: 2,000 89 and 53, 138 and 140, 500 26 and 26, 52
// and 79.
constexpr int64_t GEN_ALONE_ITEMS = 16000, GEN_ALONE_SHORT = 4000;
constexpr int GEN_SHORT_WORK = 3;   // D_ATTN_MAX of two blocks of 64 positions

// waves per SIMD that the registers leave room for
constexpr int gen_waves(int hd, int rep) { return rep <= 3 ? 7 - rep : rep == 4 ? (hd == 64 ? 4 : 3) : 2; }

template <int HD, int REP>
__global__ __launch_bounds__(256, gen_waves(HD, REP)) void k_attn_gen(GenAttnArgs a) {
  constexpr int LPK = HD / 8;     // lanes per key row
  constexpr int KPI = 64 / LPK;   // key rows per wave load
  constexpr int IT = 4;           // wave loads per block
  constexpr int KB = KPI * IT;    // keys per block
  constexpr int NW = 4;           // waves per workgroup, shares per item
  constexpr bool ALONE = REP <= 3;
  __shared__ float so_[ALONE ? NW * NW : NW][REP][HD], sm_[ALONE ? NW * NW : NW][REP], sl_[ALONE ? NW * NW : NW][REP];
  const int64_t n = a.gen_desc[D_NSEQ], sb = a.gen_desc[D_SEQ_BEGIN], tb = a.chunk_desc[D_TOK_BEGIN];
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), gk = lane / LPK, c = lane % LPK;
  const int d_q = a.n_heads * HD, d_kv = a.n_kv * HD;
  const float scale = 1.4426950408889634f / sqrtf(static_cast<float>(HD));   // log2(e) / sqrt(hd)
  const uint16_t* qkv = static_cast<const uint16_t*>(a.qkv);
  const uint16_t* kvc = static_cast<const uint16_t*>(a.kvc);
  const uint16_t* pkv = static_cast<const uint16_t*>(a.pkv);
  uint16_t* gkv = static_cast<uint16_t*>(a.gkv);
  uint16_t* out = static_cast<uint16_t*>(a.out);
  const int64_t ld = a.ld;
  const int64_t items = n * a.n_kv;
  // Where items are many, each wave takes items by itself, their shares one
  // after another: the same sums without waiting for the other waves.
  const bool is_short = a.chunk_desc[D_ATTN_MAX] > 0 && a.chunk_desc[D_ATTN_MAX] <= GEN_SHORT_WORK && a.step < 64;
  const bool alone = ALONE && items >= (is_short ? GEN_ALONE_SHORT : GEN_ALONE_ITEMS);
  const int per_wg = alone ? NW : 1;
  float (*const so)[REP][HD] = so_ + (alone ? NW * w : 0);
  float (*const sm)[REP] = sm_ + (alone ? NW * w : 0);
  float (*const sl)[REP] = sl_ + (alone ? NW * w : 0);
  auto sync = [&]() {
    if (alone) {   // LDS is in order within a wave
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    } else {
      __syncthreads();
    }
  };

  for (int64_t item = static_cast<int64_t>(blockIdx.x) * per_wg + (alone ? w : 0); item < items;
       item += static_cast<int64_t>(gridDim.x) * per_wg) {
    const int64_t i = item <= INT32_MAX ? static_cast<int32_t>(item) / a.n_kv : item / a.n_kv;
    const int kvh = static_cast<int>(item - i * a.n_kv);
    const int64_t s0 = a.cu[sb + i] - tb;
    const int own = static_cast<int>(a.cu[sb + i + 1] - a.cu[sb + i]);
    const int P = a.npre + own;   // prompt positions
    if (a.last_row && own == 0) continue;   // no own row to attend from (same for all waves of the item)
    // keys: the prompt, the earlier generated tokens, this token (last-row
    // mode: the prompt, whose last row is the query)
    const int N = a.last_row ? P : P + a.step + 1;
    const uint16_t* qrow = !a.last_row ? qkv + i * ld : (qkv ? qkv + i * a.ldq : kvc + (s0 + own - 1) * ld);
    const int kc = d_q + kvh * HD, vc = d_q + d_kv + kvh * HD;   // key / value columns of a q|k|v row
    uint16_t* gslot = a.last_row ? nullptr : gkv + (i * a.gen + a.step) * (2 * d_kv);
    if (!a.last_row && (alone || w == 0) && lane < 2 * LPK) {
      const bool isv = lane >= LPK;
      const int cc = lane % LPK;
      *reinterpret_cast<uint4*>(gslot + (isv ? d_kv : 0) + kvh * HD + cc * 8) =
          *reinterpret_cast<const uint4*>(qrow + (isv ? vc : kc) + cc * 8);
    }
    float qf[REP][8];
#pragma unroll
    for (int r = 0; r < REP; ++r) {
      const uint4 u = *reinterpret_cast<const uint4*>(qrow + (kvh * REP + r) * HD + c * 8);
      const uint32_t uw[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        qf[r][2 * e] = h2f(static_cast<uint16_t>(uw[e] & 0xFFFFu)) * scale;
        qf[r][2 * e + 1] = h2f(static_cast<uint16_t>(uw[e] >> 16)) * scale;
      }
    }
    // this lane's 16-byte pieces of key j's key and value rows
    auto rows_of = [&](int j, const uint16_t*& kp, const uint16_t*& vp) {
      const uint16_t* row;
      int ko = kc, vo = vc;
      if (j < a.npre) {
        row = pkv + static_cast<int64_t>(j) * ld;
      } else if (j < P) {
        row = kvc + (s0 + j - a.npre) * ld;
      } else if (j < P + a.step) {
        row = gkv + (i * a.gen + (j - P)) * (2 * d_kv);
        ko = kvh * HD;
        vo = d_kv + kvh * HD;
      } else {
        row = qrow;
      }
      kp = row + ko + c * 8;
      vp = row + vo + c * 8;
    };
    auto load_block = [&](int kb, uint4 (&kr)[IT], uint4 (&vr)[IT]) {
#pragma unroll
      for (int it = 0; it < IT; ++it) {
        const int j = kb + it * KPI + gk;
        kr[it] = make_uint4(0, 0, 0, 0);
        vr[it] = make_uint4(0, 0, 0, 0);
        if (j < N) {
          const uint16_t *kp, *vp;
          rows_of(j, kp, vp);
          kr[it] = *reinterpret_cast<const uint4*>(kp);
          vr[it] = *reinterpret_cast<const uint4*>(vp);
        }
      }
    };

    const int v_end = alone ? (N > (NW - 1) * KB ? NW : (N + KB - 1) / KB) : w + 1;
    for (int v = alone ? 0 : w; v < v_end; ++v) {
      float m[REP], l[REP], o[REP][8];
#pragma unroll
      for (int r = 0; r < REP; ++r) {
        m[r] = -INFINITY;
        l[r] = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) o[r][e] = 0.f;
      }
      for (int kb = v * KB; kb < N; kb += NW * KB) {
        uint4 kr[IT], vr[IT];
        load_block(kb, kr, vr);
        float s[REP][IT];
#pragma unroll
        for (int it = 0; it < IT; ++it) {
          const uint32_t uw[4] = {kr[it].x, kr[it].y, kr[it].z, kr[it].w};
          float kf[8];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            kf[2 * e] = h2f(static_cast<uint16_t>(uw[e] & 0xFFFFu));
            kf[2 * e + 1] = h2f(static_cast<uint16_t>(uw[e] >> 16));
          }
          const bool ok = kb + it * KPI + gk < N;
#pragma unroll
          for (int r = 0; r < REP; ++r) {
            float dot = 0.f;
#pragma unroll
            for (int e = 0; e < 8; ++e) dot = fmaf(qf[r][e], kf[e], dot);
            dot = dpp_add(dot, LPK);
            s[r][it] = ok ? dot : -INFINITY;
          }
        }
        float vf[IT][8];
#pragma unroll
        for (int it = 0; it < IT; ++it) {
          const uint32_t uw[4] = {vr[it].x, vr[it].y, vr[it].z, vr[it].w};
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            vf[it][2 * e] = h2f(static_cast<uint16_t>(uw[e] & 0xFFFFu));
            vf[it][2 * e + 1] = h2f(static_cast<uint16_t>(uw[e] >> 16));
          }
        }
#pragma unroll
        for (int r = 0; r < REP; ++r) {
          float mx = m[r];
#pragma unroll
          for (int it = 0; it < IT; ++it) mx = fmaxf(mx, s[r][it]);
          const float ref = mx == -INFINITY ? 0.f : mx;   // no key of this group yet: every term below is 0
          const float alpha = __builtin_amdgcn_exp2f(m[r] - ref);
          float p[IT], ps = 0.f;
#pragma unroll
          for (int it = 0; it < IT; ++it) {
            p[it] = __builtin_amdgcn_exp2f(s[r][it] - ref);   // 0 for keys past the end (score -inf)
            ps += p[it];
          }
          l[r] = l[r] * alpha + ps;
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            float acc = o[r][e] * alpha;
#pragma unroll
            for (int it = 0; it < IT; ++it) acc = fmaf(p[it], vf[it][e], acc);
            o[r][e] = acc;
          }
          m[r] = mx;
        }
      }
      // the key groups of the wave (then the shares: key 0 makes one maximum finite)
      auto add = [](float x, float y) { return x + y; };
      auto max2 = [](float x, float y) { return fmaxf(x, y); };
#pragma unroll
      for (int r = 0; r < REP; ++r) {
        const float mw = across_groups<LPK>(m[r], max2);
        const float f = mw == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m[r] - mw);
        const float lw = across_groups<LPK>(l[r] * f, add);
#pragma unroll
        for (int e = 0; e < 8; ++e) o[r][e] = across_groups<LPK>(o[r][e] * f, add);
        if (gk == 0) {
#pragma unroll
          for (int e = 0; e < 8; ++e) so[v][r][c * 8 + e] = o[r][e];
          if (c == 0) {
            sm[v][r] = mw;
            sl[v][r] = lw;
          }
        }
      }
    }
    sync();
    auto merge = [&](auto all, int shares, int first, int step) {   // two output values per thread
      for (int j = first; j < REP * HD / 2; j += step) {
        const int r = j / (HD / 2), e = (j % (HD / 2)) * 2;
        float mm = sm[0][r], ls = 0.f, o0 = 0.f, o1 = 0.f;
        auto take = [&](int v) {
          const float f = __builtin_amdgcn_exp2f(sm[v][r] - mm);   // 0 for a share without keys
          ls = fmaf(sl[v][r], f, ls);
          o0 = fmaf(so[v][r][e], f, o0);
          o1 = fmaf(so[v][r][e + 1], f, o1);
        };
        if (decltype(all)::value) {
#pragma unroll
          for (int v = 1; v < NW; ++v) mm = fmaxf(mm, sm[v][r]);
#pragma unroll
          for (int v = 0; v < NW; ++v) take(v);
        } else {
          for (int v = 1; v < shares; ++v) mm = fmaxf(mm, sm[v][r]);
          for (int v = 0; v < shares; ++v) take(v);
        }
        const float inv = 1.0f / ls;
        *reinterpret_cast<uint32_t*>(out + i * d_q + (kvh * REP + r) * HD + e) =
            f2act(o0 * inv, a.out_act) | (static_cast<uint32_t>(f2act(o1 * inv, a.out_act)) << 16);
      }
    };
    if (alone)
      merge(std::false_type{}, v_end, lane, 64);   // shares without keys add nothing
    else
      merge(std::true_type{}, NW, static_cast<int>(threadIdx.x), 64 * NW);
    sync();   // the partial states are read before the next item writes them
  }
}

hipError_t launch_attention_gen(const GenAttnArgs& a, hipStream_t s) {
  if (a.n_kv <= 0 || a.n_heads % a.n_kv || a.npre < 0 || (a.npre > 0 && !a.pkv) || a.out_act == ACT_F32 ||
      (!a.last_row && (a.step < 0 || a.step >= a.gen || !a.gkv || !a.qkv)))
    return hipErrorInvalidValue;
  const int rep = a.n_heads / a.n_kv;
  const dim3 grid(grid_for(a.seq_ub * a.n_kv, 1, 16384)), block(256);
#define AIQ_GEN_ATTN(HD_)                                                          \
  switch (rep) {                                                                   \
    case 1: hipLaunchKernelGGL((k_attn_gen<HD_, 1>), grid, block, 0, s, a); break; \
    case 2: hipLaunchKernelGGL((k_attn_gen<HD_, 2>), grid, block, 0, s, a); break; \
    case 3: hipLaunchKernelGGL((k_attn_gen<HD_, 3>), grid, block, 0, s, a); break; \
    case 4: hipLaunchKernelGGL((k_attn_gen<HD_, 4>), grid, block, 0, s, a); break; \
    case 8: hipLaunchKernelGGL((k_attn_gen<HD_, 8>), grid, block, 0, s, a); break; \
    default: return hipErrorInvalidValue;                                          \
  }
  if (a.hd == 64) {
    AIQ_GEN_ATTN(64)
  } else if (a.hd == 128) {
    AIQ_GEN_ATTN(128)
  } else {
    return hipErrorInvalidValue;
  }
#undef AIQ_GEN_ATTN
  return hipGetLastError();
}

// ------------------------------------------------------------------ final norm of the step rows
// Normalised in fp32, then rounded: the head's 16-bit operand keeps its range
// and its bits whatever the residual's size (x * g alone overflows fp16 above
// 65,504 and loses bits below 6e-5).
__global__ __launch_bounds__(256) void k_norm_rows(const int64_t* gd, const float* x, const float* g, int32_t d,
                                                   float eps, uint16_t* hf, int32_t act) {
  const int64_t n = gd[D_NSEQ];
  const int lane = threadIdx.x & 63;
  const int64_t wave = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6;
  const int64_t n_waves = ((int64_t)gridDim.x * blockDim.x) >> 6;
  for (int64_t i = wave; i < n; i += n_waves) {
    const float* xr = x + i * d;
    float ss = 0.f;
    for (int c = lane; c < d; c += 64) ss += xr[c] * xr[c];
    ss = wave_sum_g(ss);
    const float r = 1.0f / sqrtf(ss / static_cast<float>(d) + eps);
    for (int c = lane; c < d; c += 64) hf[i * d + c] = f2act(xr[c] * r * g[c], act);
  }
}

hipError_t launch_norm_rows(const int64_t* gen_desc, const float* x, const float* g, int32_t d, float eps, void* hf,
                            int32_t act, int64_t seq_ub, hipStream_t s) {
  if (act == ACT_F32) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_norm_rows, dim3(grid_for(seq_ub, 4, 4096)), dim3(256), 0, s, gen_desc, x, g, d, eps,
                     static_cast<uint16_t*>(hf), act);
  return hipGetLastError();
}

// ------------------------------------------------------------------ the next token and its embedding
// The head GEMM leaves, per row, the maximum and its column over every 64
// columns (lowest column on ties); a wave per row picks the largest, again
// the lowest column among equals, records the token and, but in the last step
// (also for rows that have ended, whose tokens are pads), writes the token's embedding for the next one (x, the
// first norm's operand h = x * g, its row scale, the position): one launch where the
// argmax and the embedding took 5 us each.
__global__ __launch_bounds__(256) void k_gen_next(GenNextArgs a) {
  const int64_t rows = *a.cnt, sb = a.gen_desc[D_SEQ_BEGIN];
  const int n_chunk = a.vocab / 64;
  const int ea = a.wdtype == AIQ_F16 ? ACT_F16 : ACT_BF16;
  const int lane = threadIdx.x & 63;
  const int64_t wave = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6;
  const int64_t n_waves = ((int64_t)gridDim.x * blockDim.x) >> 6;
  for (int64_t r = wave; r < rows; r += n_waves) {
    const int2* pr = static_cast<const int2*>(a.part) + r * n_chunk;
    float best = -INFINITY;
    int32_t bi = INT32_MAX;
    for (int c = lane; c < n_chunk; c += 64) {   // ascending columns: strict > keeps each lane's first maximum
      const int2 p = pr[c];
      const float v = __int_as_float(p.x);
      if (v > best) {
        best = v;
        bi = p.y;
      }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      const float ov = __shfl_xor(best, o);
      const int32_t oi = __shfl_xor(bi, o);
      if (ov > best || (ov == best && oi < bi)) {
        best = ov;
        bi = oi;
      }
    }
    if (bi == INT32_MAX) bi = 0;   // no finite maximum (every logit NaN or -inf)
    const int64_t i = a.row0 + r;
    if (lane == 0) {
      const bool ended = a.done[i] != 0;
      a.gen[(sb + i) * a.G + a.step] = ended ? a.pad : bi;
      if (!ended && bi == a.eos) a.done[i] = 1;
    }
    if (a.step + 1 == a.G) continue;
    if (lane == 0) a.pos[i] = a.npre + static_cast<int32_t>(a.cu[sb + i + 1] - a.cu[sb + i]) + a.step;
    const int d = a.d;
    const uint16_t* er = static_cast<const uint16_t*>(a.emb) + static_cast<int64_t>(bi) * d;
    float* xr = a.x + i * d;
    uint16_t* hr = static_cast<uint16_t*>(a.h) + i * d;
    float ssq = 0.f;
    for (int c = lane * 4; c < d; c += 256) {
      const uint2 v = *reinterpret_cast<const uint2*>(er + c);
      float4 o;
      o.x = act2f(static_cast<uint16_t>(v.x & 0xFFFFu), ea);
      o.y = act2f(static_cast<uint16_t>(v.x >> 16), ea);
      o.z = act2f(static_cast<uint16_t>(v.y & 0xFFFFu), ea);
      o.w = act2f(static_cast<uint16_t>(v.y >> 16), ea);
      *reinterpret_cast<float4*>(xr + c) = o;
      const float4 gv = *reinterpret_cast<const float4*>(a.g + c);
      uint2 hv;
      hv.x = f2act(o.x * gv.x, a.h_act) | (static_cast<uint32_t>(f2act(o.y * gv.y, a.h_act)) << 16);
      hv.y = f2act(o.z * gv.z, a.h_act) | (static_cast<uint32_t>(f2act(o.w * gv.w, a.h_act)) << 16);
      *reinterpret_cast<uint2*>(hr + c) = hv;
      ssq += (o.x * o.x + o.y * o.y) + (o.z * o.z + o.w * o.w);
    }
    ssq = wave_sum_g(ssq);
    if (lane == 0) a.rs[i] = 1.0f / sqrtf(ssq / static_cast<float>(d) + a.eps);
  }
}

hipError_t launch_gen_next(const GenNextArgs& a, hipStream_t s) {
  if (a.vocab % 64 || (a.wdtype != AIQ_BF16 && a.wdtype != AIQ_F16) || a.h_act == ACT_F32 || a.d % 4)
    return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_gen_next, dim3(grid_for(GEN_HEAD_ROWS, 4, 1024)), dim3(256), 0, s, a);
  return hipGetLastError();
}

// ------------------------------------------------------------------ LIKE over the generated tokens
// Wave per selected row: the generated length (through the first end token),
// then every start position tested by one lane.
__global__ __launch_bounds__(256) void k_gen_like(const int32_t* gen, const int64_t* n_ptr, int32_t G, int32_t eos,
                                                  LikePattern pat, int32_t* label) {
  const int64_t n = *n_ptr;
  const int lane = threadIdx.x & 63;
  const int64_t wave = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6;
  const int64_t n_waves = ((int64_t)gridDim.x * blockDim.x) >> 6;
  for (int64_t i = wave; i < n; i += n_waves) {
    const int32_t* gr = gen + i * G;
    int glen = G;
    if (eos >= 0) {
      for (int c = 0; c < G; c += 64) {
        const uint64_t b = __ballot(c + lane < G && gr[c + lane] == eos);
        if (b) {
          glen = c + __builtin_ctzll(b) + 1;
          break;
        }
      }
    }
    bool hit = false;
    if (pat.n == 0) {
      hit = true;
    } else {
      for (int s = lane; s + pat.n <= glen; s += 64) {
        bool ok = true;
        for (int q = 0; q < pat.n && ok; ++q) ok = gr[s + q] == pat.tok[q];
        hit = hit || ok;
      }
      hit = __ballot(hit) != 0;
    }
    if (lane == 0) label[i] = hit ? 1 : 0;
  }
}

hipError_t launch_gen_like(const int32_t* gen, const int64_t* n_ptr, int64_t n_ub, int32_t G, int32_t eos,
                           const LikePattern& pat, int32_t* label, hipStream_t s) {
  if (pat.n < 0 || pat.n > AIQ_MAX_LIKE || G <= 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_gen_like, dim3(grid_for(n_ub, 4, 4096)), dim3(256), 0, s, gen, n_ptr, G, eos, pat, label);
  return hipGetLastError();
}

__global__ void k_copy_rows_i32(const int32_t* src, const int64_t* n_ptr, int32_t per_row, int32_t* dst,
                                int64_t cap_rows) {
  int64_t rows = *n_ptr;
  if (rows > cap_rows) rows = cap_rows;
  const int64_t total = rows * per_row;
  for (int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; j < total; j += (int64_t)gridDim.x * blockDim.x)
    dst[j] = src[j];
}

hipError_t launch_copy_rows_i32(const int32_t* src, const int64_t* n_ptr, int64_t n_ub, int32_t per_row,
                                int32_t* dst, int64_t cap_rows, hipStream_t s) {
  const int64_t ub = (n_ub < cap_rows ? n_ub : cap_rows) * per_row;
  hipLaunchKernelGGL(k_copy_rows_i32, dim3(grid_for(ub, 256, 4096)), dim3(256), 0, s, src, n_ptr, per_row, dst,
                     cap_rows);
  return hipGetLastError();
}

}  // namespace aiq
