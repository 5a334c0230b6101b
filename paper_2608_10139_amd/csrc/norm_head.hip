// RMSNorm of the residual stream, and the last-position label head.
//
// The semantic decision reads only the last position's logits of each row
// and only the label columns (Figure 2: logits[:, -1, :], then the Yes / No
// columns compared on chip).  The head therefore never forms the [tokens,
// vocab] logits: one workgroup per sequence takes the last token's residual row
// in fp32, its norm and K dot products with the label rows of the LM head.
#include "aiq_internal.h"
#include "dev_util.h"

namespace aiq {

static int grid_for(int64_t n, int per_block, int cap) {
  int64_t g = (n + per_block - 1) / per_block;
  if (g < 1) g = 1;
  if (g > cap) g = cap;
  return static_cast<int>(g);
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}


// ------------------------------------------------------------------ residual add + RMSNorm
// One wave per row.  With a pending projection output `delta` the residual
// stream is updated first (x += delta, fp32, written back), then
// out = x / sqrt(mean(x^2) + eps) * g.  The sum of squares is reduced in a
// fixed order inside the row, so a row's result does not depend on which
// other rows share the launch.
// MAXV: float4 pieces per lane (rows of up to 256 * MAXV floats); a small one for
// narrow models keeps 16 unrolled, mostly empty pieces out of the launch (5,392 rows of
// d 128: 7.2 us with 16, 5.3 with 2).
template <int MAXV>
__global__ __launch_bounds__(256) void k_rmsnorm(const int64_t* desc, float* x, const float* delta, const float* g,
                                                 int32_t d, float eps, void* out, int32_t out_act) {
  const int64_t nt = desc[D_NTOK];
  const int lane = threadIdx.x & 63;
  const int64_t wave = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6;
  const int64_t n_waves = ((int64_t)gridDim.x * blockDim.x) >> 6;
  const int nv = d >> 2;
  for (int64_t t = wave; t < nt; t += n_waves) {
    float4* xr = reinterpret_cast<float4*>(x + t * d);
    float4 v[MAXV];
    float ss = 0.f;
#pragma unroll
    for (int j = 0; j < MAXV; ++j) {
      const int c = lane + 64 * j;
      if (c < nv) {
        float4 a = xr[c];
        if (delta) {
          const float4 b = reinterpret_cast<const float4*>(delta + t * d)[c];
          a.x += b.x; a.y += b.y; a.z += b.z; a.w += b.w;
          xr[c] = a;
        }
        v[j] = a;
        ss += a.x * a.x + a.y * a.y + a.z * a.z + a.w * a.w;
      }
    }
    ss = wave_sum(ss);
    const float r = 1.0f / sqrtf(ss / static_cast<float>(d) + eps);
    const float4* gr = reinterpret_cast<const float4*>(g);
#pragma unroll
    for (int j = 0; j < MAXV; ++j) {
      const int c = lane + 64 * j;
      if (c < nv) {
        const float4 a = v[j], w = gr[c];
        if (out_act != ACT_F32) {
          uint2 p;
          p.x = f2act(a.x * r * w.x, out_act) | (static_cast<uint32_t>(f2act(a.y * r * w.y, out_act)) << 16);
          p.y = f2act(a.z * r * w.z, out_act) | (static_cast<uint32_t>(f2act(a.w * r * w.w, out_act)) << 16);
          reinterpret_cast<uint2*>(static_cast<uint16_t*>(out) + t * d)[c] = p;
        } else {
          reinterpret_cast<float4*>(static_cast<float*>(out) + t * d)[c] =
              make_float4(a.x * r * w.x, a.y * r * w.y, a.z * r * w.z, a.w * r * w.w);
        }
      }
    }
  }
}

hipError_t launch_rmsnorm(const int64_t* desc, float* x, const float* delta, const float* g, int32_t d,
                          float eps, void* out, int32_t out_act, int64_t t_cap, hipStream_t s) {
  if (d > 64 * 4 * 16) return hipErrorInvalidValue;
  const dim3 grid(grid_for(t_cap, 4, 4096));
  if (d <= 64 * 4 * 2)
    hipLaunchKernelGGL(k_rmsnorm<2>, grid, dim3(256), 0, s, desc, x, delta, g, d, eps, out, out_act);
  else
    hipLaunchKernelGGL(k_rmsnorm<16>, grid, dim3(256), 0, s, desc, x, delta, g, d, eps, out, out_act);
  return hipGetLastError();
}

// ------------------------------------------------------------------ row scale
// The RMSNorm scale of each token from the per-slice sums of squares that the
// residual projection wrote, added in slice order.  A block takes 128 tokens:
// their rows of sums come in with coalesced 16-byte loads into LDS (rows
// padded by one float: conflict-free), then one thread per token adds its row
// (rows wider than RS_MAX_PART: each thread reads its row directly).
constexpr int RS_TOK = 128, RS_MAX_PART = 64;

__global__ __launch_bounds__(256) void k_row_scale(const int64_t* desc, const float* ssp, int32_t n_part, int32_t d,
                                                   float eps, float* rs) {
  __shared__ float part[RS_TOK * (RS_MAX_PART + 1)];
  const int64_t nt = desc[D_NTOK];
  if (n_part > RS_MAX_PART || n_part % 4) {   // wide models: thread per token straight from memory
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < nt; t += (int64_t)gridDim.x * blockDim.x) {
      const float* p = ssp + t * n_part;
      float ss = 0.f;
      for (int k = 0; k < n_part; ++k) ss += p[k];
      rs[t] = 1.0f / sqrtf(ss / static_cast<float>(d) + eps);
    }
    return;
  }
  const int stride = n_part + 1;
  const int q4 = n_part / 4;   // 16-byte pieces per token
  for (int64_t t0 = static_cast<int64_t>(blockIdx.x) * RS_TOK; t0 < nt; t0 += static_cast<int64_t>(gridDim.x) * RS_TOK) {
    const int ntok = nt - t0 < RS_TOK ? static_cast<int>(nt - t0) : RS_TOK;
    const float4* src = reinterpret_cast<const float4*>(ssp + t0 * n_part);
    for (int e = threadIdx.x; e < ntok * q4; e += blockDim.x) {
      const float4 v = src[e];
      float* dst = part + (e / q4) * stride + (e % q4) * 4;
      dst[0] = v.x;
      dst[1] = v.y;
      dst[2] = v.z;
      dst[3] = v.w;
    }
    __syncthreads();
    if (threadIdx.x < ntok) {
      const float* p = part + threadIdx.x * stride;
      float ss = 0.f;
      for (int k = 0; k < n_part; ++k) ss += p[k];
      rs[t0 + threadIdx.x] = 1.0f / sqrtf(ss / static_cast<float>(d) + eps);
    }
    __syncthreads();
  }
}

hipError_t launch_row_scale(const int64_t* desc, const float* ssp, int32_t n_part, int32_t d, float eps,
                            float* rs, int64_t t_cap, hipStream_t s) {
  if (n_part <= 0) return hipErrorInvalidValue;
  const int per_block = (n_part > RS_MAX_PART || n_part % 4) ? 256 : RS_TOK;
  hipLaunchKernelGGL(k_row_scale, dim3(grid_for(t_cap, per_block, 4096)), dim3(256), 0, s, desc, ssp, n_part, d, eps,
                     rs);
  return hipGetLastError();
}

// ------------------------------------------------------------------ label head + decision
// Workgroup per sequence of the chunk: one pass over the row for its sum of
// squares and its unscaled dot products with the label rows (float4 pieces; the
// scale 1 / rms is applied to the sums), a second over the row for hf_out.
// With one wave per sequence and 4-byte loads in a chain per label the head of 8
// sequences of d 3072 took 55 us; this takes 10 (128 of d 2048: 45, 9).
// NW waves, as many as a row's float4 pieces occupy (at most four; idle ones cost
// many sequences their barriers: 100,000 of d 128 268 us with four, 20,000 of d 512 56 and 30).
// label_out / logits_out are indexed by the global
// sequence number (seq_begin + local index).
template <int NW>
__global__ __launch_bounds__(64 * NW) void k_head(HeadArgs a) {
  __shared__ float red[NW][AIQ_MAX_LABELS + 1];
  const int64_t tb = a.desc[D_TOK_BEGIN], sb = a.desc[D_SEQ_BEGIN], ns = a.desc[D_NSEQ];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int d = a.d;
  const bool w16 = a.wdtype == AIQ_BF16 || a.wdtype == AIQ_F16;
  const int wa = a.wdtype == AIQ_F16 ? ACT_F16 : ACT_BF16;
  for (int64_t i = blockIdx.x; i < ns; i += gridDim.x) {
    const int64_t gi = sb + i;
    const int64_t c1 = a.cu[gi + 1];
    // no own token: the shared prefix's last token, else every logit is 0
    const bool no_own = c1 == a.cu[gi];
    const bool empty = no_own && !a.x_pre;
    const bool pre = no_own && a.x_pre;
    const int64_t last = no_own ? 0 : (a.x_compact ? i : c1 - 1 - tb);
    const float* xr = pre ? a.x_pre : a.x + last * d;
    const float* dr = (a.delta && !pre) ? a.delta + last * d : nullptr;   // last layer's pending output
    // an empty sequence reads no row: its normalised state is 0
    auto xv = [&](int c) {
      float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
      if (empty) return v;
      v = *reinterpret_cast<const float4*>(xr + c);
      if (dr) {
        const float4 u = *reinterpret_cast<const float4*>(dr + c);
        v.x += u.x; v.y += u.y; v.z += u.z; v.w += u.w;
      }
      return v;
    };
    float ss = 0.f, acc[AIQ_MAX_LABELS];
#pragma unroll
    for (int k = 0; k < AIQ_MAX_LABELS; ++k) acc[k] = 0.f;
    for (int c = t * 4; c < d; c += 256 * NW) {
      const float4 x = xv(c), g = *reinterpret_cast<const float4*>(a.g + c);
      ss += (x.x * x.x + x.y * x.y) + (x.z * x.z + x.w * x.w);
#pragma unroll
      for (int k = 0; k < AIQ_MAX_LABELS; ++k) {
        if (k >= a.n_labels) break;
        float4 wv;
        const int64_t wo = static_cast<int64_t>(a.labels[k]) * d + c;
        if (w16) {
          const uint2 u = *reinterpret_cast<const uint2*>(static_cast<const uint16_t*>(a.lm_head) + wo);
          wv = make_float4(act2f(static_cast<uint16_t>(u.x & 0xFFFFu), wa), act2f(static_cast<uint16_t>(u.x >> 16), wa),
                           act2f(static_cast<uint16_t>(u.y & 0xFFFFu), wa), act2f(static_cast<uint16_t>(u.y >> 16), wa));
        } else {
          wv = *reinterpret_cast<const float4*>(static_cast<const float*>(a.lm_head) + wo);
        }
        acc[k] += ((x.x * g.x) * wv.x + (x.y * g.y) * wv.y) + ((x.z * g.z) * wv.z + (x.w * g.w) * wv.w);
      }
    }
    ss = wave_sum(ss);
#pragma unroll
    for (int k = 0; k < AIQ_MAX_LABELS; ++k) {
      if (k >= a.n_labels) break;
      acc[k] = wave_sum(acc[k]);
    }
    if (NW > 1) {
      if (lane == 0) {
        red[w][AIQ_MAX_LABELS] = ss;
#pragma unroll
        for (int k = 0; k < AIQ_MAX_LABELS; ++k) {
          if (k >= a.n_labels) break;
          red[w][k] = acc[k];
        }
      }
      __syncthreads();
      auto total = [&](int k) {
        return NW == 2 ? red[0][k] + red[1][k] : (red[0][k] + red[1][k]) + (red[NW - 2][k] + red[NW - 1][k]);
      };
      ss = total(AIQ_MAX_LABELS);
#pragma unroll
      for (int k = 0; k < AIQ_MAX_LABELS; ++k) {
        if (k >= a.n_labels) break;
        acc[k] = total(k);
      }
    }
    const float r = empty ? 0.f : 1.0f / sqrtf(ss / static_cast<float>(d) + a.eps);
    if (a.hf_out) {
      for (int c = t * 4; c < d; c += 256 * NW) {
        const float4 x = xv(c), g = *reinterpret_cast<const float4*>(a.g + c);
        const float4 o = make_float4(x.x * r * g.x, x.y * r * g.y, x.z * r * g.z, x.w * r * g.w);
        if (a.hf_act != ACT_F32) {
          uint2 p;
          p.x = f2act(o.x, a.hf_act) | (static_cast<uint32_t>(f2act(o.y, a.hf_act)) << 16);
          p.y = f2act(o.z, a.hf_act) | (static_cast<uint32_t>(f2act(o.w, a.hf_act)) << 16);
          *reinterpret_cast<uint2*>(static_cast<uint16_t*>(a.hf_out) + i * d + c) = p;
        } else {
          *reinterpret_cast<float4*>(static_cast<float*>(a.hf_out) + i * d + c) = o;
        }
      }
    }
    if (t == 0 && (a.logits_out || a.label_out)) {
      float lg[AIQ_MAX_LABELS];
#pragma unroll
      for (int k = 0; k < AIQ_MAX_LABELS; ++k) {
        if (k >= a.n_labels) break;
        lg[k] = acc[k] * r;
        if (a.logits_out) a.logits_out[gi * a.n_labels + k] = lg[k];
      }
      if (a.label_out) {
        int32_t lab;
        if (a.decision == AIQ_DECIDE_BINARY_GT) {
          lab = lg[0] > lg[1] ? 1 : 0;
        } else {
          int best = 0;
          float bv = lg[0];
#pragma unroll
          for (int k = 1; k < AIQ_MAX_LABELS; ++k) {
            if (k >= a.n_labels) break;
            if (lg[k] > bv) {
              bv = lg[k];
              best = k;
            }
          }
          lab = a.labels[best];
        }
        a.label_out[gi] = lab;
      }
    }
    if (NW > 1) __syncthreads();   // the partial sums are read before the next sequence writes them
  }
}

hipError_t launch_head(const HeadArgs& a, hipStream_t s) {
  if (a.d % 4) return hipErrorInvalidValue;
  if (a.d <= 256)
    hipLaunchKernelGGL(k_head<1>, dim3(grid_for(a.seq_ub, 1, 16384)), dim3(64), 0, s, a);
  else if (a.d <= 512)
    hipLaunchKernelGGL(k_head<2>, dim3(grid_for(a.seq_ub, 1, 8192)), dim3(128), 0, s, a);
  else
    hipLaunchKernelGGL(k_head<4>, dim3(grid_for(a.seq_ub, 1, 4096)), dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace aiq
