// ccq_prep.hip -- per-layer pre-processing of the raw queries and keys (Alg. 1:
// the l2 normalisation of Q and K and the gate Lambda = sigma(Q W_lambda^T + b_lambda)
// from the query before the head split; Eq. clean for the gate).
//
// Each wave takes TPW tokens (four, or one where there are few): it requests their whole q and k rows at once
// (16-byte pieces, consecutive lanes along the row), reduces each head's
// squared norms over the aligned lane group holding that head and writes the
// normalised pieces; then every gate's partial dot products
// z[h'] += W[h'][j] q[j] over the lane's pieces, each piece of W read from LDS
// once for the wave's tokens; the H partial dots are reduced over the wave and
// lane h' writes lambda[h'].  Without output rows (q and k
// null) the kernel writes the row scales 1 / max(|x|, 1e-12) instead, for a
// forward that normalises as it stages the raw rows.  W (H x H dk, fp32) is staged
// in LDS once per workgroup and shared by its 4 TPW tokens.  A wave reads each raw row before it writes the
// normalised one, so the outputs may overwrite the inputs.
#include "ccq_device.h"
#include "ccq_kernels.h"

namespace ccq {

// Sum over aligned groups of N consecutive lanes (N = 8, 16, 32), every lane
// receiving its group's sum.
template <int N>
__device__ __forceinline__ float lane_group_sum(float x) {
#pragma unroll
  for (int off = 1; off < N; off <<= 1) x += __shfl_xor(x, off);
  return x;
}

// A token's row is one long chain (request, norms over lane groups, gates, sums
// over the wave), so with few tokens a wave's own time is what counts: one token
// per wave, and the rows requested ahead of the staging of W (AHEAD).
template <typename T, int DK, int HMAX, int TPW, bool AHEAD>
__global__ __launch_bounds__(kThreads) void prep_kernel(const PrepArgs a) {
  constexpr int kPrepTokens = 4 * TPW;  // tokens per workgroup
  extern __shared__ float sW[];  // [H][H * DK], each row split in half-pieces (below)
  constexpr int PPH = DK / 8;    // 8-element pieces per head row
  constexpr int NPMAX = 4;       // pieces per lane and token (H * DK <= 2048 when supported)
  typedef T v8 __attribute__((ext_vector_type(8)));
  const int H = a.H, E = H * DK, NP = E / 8;
  const int w = wave_id(), l = lane_id();
  const long long ntok = (long long)a.B * a.T;
  const T* qr = static_cast<const T*>(a.q_raw);
  const T* kr = static_cast<const T*>(a.k_raw);
  T* qo = static_cast<T*>(a.q);
  T* ko = static_cast<T*>(a.k);
  // every piece of the wave's tokens requested at once, ahead of W_lambda or after it
  v8 qa[TPW][NPMAX], ka[TPW][NPMAX];
  auto request = [&] {
#pragma unroll
    for (int tt = 0; tt < TPW; ++tt) {
      const long long tok = (long long)blockIdx.x * kPrepTokens + w * TPW + tt;
#pragma unroll
      for (int i = 0; i < NPMAX; ++i) {
        const int p = l + 64 * i;
        if (tok < ntok && p < NP) {
          qa[tt][i] = *reinterpret_cast<const v8*>(qr + (size_t)tok * E + 8 * p);
          ka[tt][i] = *reinterpret_cast<const v8*>(kr + (size_t)tok * E + 8 * p);
        }
      }
    }
  };
  if constexpr (AHEAD) request();
  {  // W_lambda into LDS: every 16-byte piece requested before any is stored
    constexpr int NW4 = (int)(kPrepMaxLds / 16 / kThreads);
    const int n4 = H * E / 4;
    f32x4 wv[NW4];
#pragma unroll
    for (int u = 0; u < NW4; ++u) {
      const int i4 = threadIdx.x + kThreads * u;
      if (i4 < n4) wv[u] = reinterpret_cast<const f32x4*>(a.w)[i4];
    }
    // row g, features 8 p .. 8 p + 3 at g E + 4 p and 8 p + 4 .. 8 p + 7 at
    // g E + E / 2 + 4 p: a lane's two 16-byte reads of its piece p then sit
    // next to those of the neighbouring lanes (no bank conflicts)
#pragma unroll
    for (int u = 0; u < NW4; ++u) {
      const int i4 = threadIdx.x + kThreads * u;
      if (i4 < n4) {
        const int g = i4 / (E / 4), r = i4 % (E / 4);
        reinterpret_cast<f32x4*>(sW)[(g * E + (r & 1) * (E / 2)) / 4 + (r >> 1)] = wv[u];
      }
    }
  }
  __syncthreads();
  if constexpr (!AHEAD) request();
  // norms of every token's head rows; normalised rows (or the row scales) out
#pragma unroll
  for (int tt = 0; tt < TPW; ++tt) {
    const long long tok = (long long)blockIdx.x * kPrepTokens + w * TPW + tt;
    if (tok >= ntok) break;
    const size_t base = (size_t)tok * E;
#pragma unroll
    for (int i = 0; i < NPMAX; ++i) {
      const int p = l + 64 * i;
      float qf[8], kf[8], qq = 0.f, kk = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        qf[e] = p < NP ? f32(qa[tt][i][e]) : 0.f;
        kf[e] = p < NP ? f32(ka[tt][i][e]) : 0.f;
        qq += qf[e] * qf[e];
        kk += kf[e] * kf[e];
      }
      // the lanes of one head row are an aligned group of PPH (or all 64 when PPH > 64)
      qq = lane_group_sum<(PPH < 64 ? PPH : 64)>(qq);
      kk = lane_group_sum<(PPH < 64 ? PPH : 64)>(kk);
      if (p < NP) {
        const float iq = 1.f / fmaxf(sqrtf(qq), 1e-12f), ik = 1.f / fmaxf(sqrtf(kk), 1e-12f);
        if (qo) {
          v8 yq, yk;
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            yq[e] = to<T>(qf[e] * iq);
            yk[e] = to<T>(kf[e] * ik);
          }
          *reinterpret_cast<v8*>(qo + base + 8 * p) = yq;
          *reinterpret_cast<v8*>(ko + base + 8 * p) = yk;
        } else if (p % PPH == 0) {  // the row scales instead, from the head's first lane
          a.rq[(size_t)tok * H + p / PPH] = iq;
          a.rk[(size_t)tok * H + p / PPH] = ik;
        }
      }
    }
  }
  // the gates: every W piece read from LDS serves all TPW tokens of the wave
  float z[TPW][HMAX];
#pragma unroll
  for (int tt = 0; tt < TPW; ++tt)
#pragma unroll
    for (int g = 0; g < HMAX; ++g) z[tt][g] = 0.f;
#pragma unroll
  for (int i = 0; i < NPMAX; ++i) {
    const int p = l + 64 * i;
    if (p < NP) {
      float qf[TPW][8];
#pragma unroll
      for (int tt = 0; tt < TPW; ++tt)
#pragma unroll
        for (int e = 0; e < 8; ++e) qf[tt][e] = f32(qa[tt][i][e]);
#pragma unroll
      for (int g = 0; g < HMAX; ++g) {
        if (g < H) {
          const f32x4 w0 = *reinterpret_cast<const f32x4*>(sW + g * E + 4 * p);
          const f32x4 w1 = *reinterpret_cast<const f32x4*>(sW + g * E + E / 2 + 4 * p);
#pragma unroll
          for (int tt = 0; tt < TPW; ++tt)
#pragma unroll
            for (int e = 0; e < 4; ++e) z[tt][g] += w0[e] * qf[tt][e] + w1[e] * qf[tt][4 + e];
        }
      }
    }
  }
  // sums over the wave of the TPW x HMAX partial dots by a reduce-scatter
  // butterfly: at each step a lane keeps half of its values, adds its
  // partner's copy of them and hands over the other half, so that after
  // log2(TPW HMAX) steps lane l holds the partial sum of value l % (TPW HMAX)
  // over the lanes that share its low bits; where 64 lanes exceed the values,
  // the exchanges between those lanes complete the sum
  constexpr int NZ = TPW * HMAX;
  static_assert(NZ <= 64 && (NZ & (NZ - 1)) == 0, "at most one value per lane after the butterfly");
  float zz[NZ];
#pragma unroll
  for (int tt = 0; tt < TPW; ++tt)
#pragma unroll
    for (int g = 0; g < HMAX; ++g) zz[tt * HMAX + g] = z[tt][g];
#pragma unroll
  for (int half = NZ / 2; half >= 1; half >>= 1) {
    // lanes with bit `half` set keep the upper half of their current values
    const bool up = (l & half) != 0;
#pragma unroll
    for (int j = 0; j < half; ++j) {
      const float mine = up ? zz[half + j] : zz[j];
      const float other = up ? zz[j] : zz[half + j];
      zz[j] = mine + __shfl_xor(other, half);
    }
  }
#pragma unroll
  for (int off = NZ; off < 64; off <<= 1) zz[0] += __shfl_xor(zz[0], off);
  // lane l now holds value l % NZ (token l / HMAX, gate l % HMAX), summed over the wave
  if (l < NZ) {
    const int tt = l / HMAX, g = l % HMAX;
    const long long tok = (long long)blockIdx.x * kPrepTokens + w * TPW + tt;
    if (g < H && tok < ntok) a.lam[(size_t)tok * H + g] = 1.f / (1.f + __expf(-(zz[0] + a.b[g])));
  }
}

namespace {
template <typename T, int DK>
hipError_t run_prep(const PrepArgs& a, hipStream_t st) {
  const long long ntok = (long long)a.B * a.T;
  if (ntok == 0 || a.H == 0) return hipSuccess;
  const size_t lds = (size_t)a.H * a.H * DK * sizeof(float);
  // One token per wave while the workgroups of four tokens fit the chip at once
  // (two per compute unit by the LDS of W_lambda): us with one against four at 2048
  // tokens 20.2 / 22.9 (8 heads of 256), 18.5 / 19.5 (11 of 128), 15.8 / 16.2 (14 of
  // 64), at 2304 29.6 / 23.4, 27.5 / 19.7, 19.2 / 16.3.  With 16 heads, whose W_lambda
  // is the largest beside a row, only while a compute unit stages it once: 16 of
  // 64, 14.8 / 16.7 at 1024 tokens, 17.1 / 16.7 at 1100, 18.0 / 17.2 at 2048 (fp32
  // 19.3 / 18.8).
  if (ntok <= (a.H > 14 ? 4 * 256 : 4 * 512)) {
    hipLaunchKernelGGL((prep_kernel<T, DK, kPrepMaxHeads, 1, true>), dim3((unsigned)((ntok + 3) / 4)), dim3(kThreads),
                       lds, st, a);
    return hipGetLastError();
  }
  // With four, the rows ahead of W_lambda only where there is a second round of
  // workgroups: loads return in order, so W_lambda waits for the rows (8 heads of
  // 256: 30.1 after, 31.0 ahead at 4500 tokens, 66.6 after, 65.4 ahead at 16384; 16 of
  // 64: 22.1 / 22.4 and 47.1 / 45.3).
  const dim3 grid((unsigned)((ntok + 15) / 16));
  if (ntok <= 16 * 512)
    hipLaunchKernelGGL((prep_kernel<T, DK, kPrepMaxHeads, 4, false>), grid, dim3(kThreads), lds, st, a);
  else
    hipLaunchKernelGGL((prep_kernel<T, DK, kPrepMaxHeads, 4, true>), grid, dim3(kThreads), lds, st, a);
  return hipGetLastError();
}
template <typename T>
hipError_t prep_dispatch(const PrepArgs& a, hipStream_t st) {
  switch (a.dk) {
    case 64: return run_prep<T, 64>(a, st);
    case 128: return run_prep<T, 128>(a, st);
    case 256: return run_prep<T, 256>(a, st);
  }
  return hipErrorInvalidValue;
}
}  // namespace

bool prep_supported(int H, int dk) {
  // H * dk <= 2048 follows from the LDS bound for H >= 8; it is checked for
  // fewer heads too (at most four 8-element pieces per lane and token)
  return (dk == 64 || dk == 128 || dk == 256) && H >= 1 && H <= kPrepMaxHeads &&
         (size_t)H * H * dk * sizeof(float) <= kPrepMaxLds && H * dk <= 2048;
}

hipError_t launch_prep(const PrepArgs& a, bool is_bf16, hipStream_t st) {
  return is_bf16 ? prep_dispatch<bf16_t>(a, st) : prep_dispatch<float>(a, st);
}

}  // namespace ccq
