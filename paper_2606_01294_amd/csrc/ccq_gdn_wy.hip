// ccq_gdn_wy.hip -- Gated DeltaNet state pass in WY form (bf16).
//
// The chunk's corrected values are affine in the state it is entered with:
//
//   U = Tm diag(beta) (V - diag(e^gamma) K S_r^T) = Tb V + W S_r^T,
//   Tb = Tm diag(beta),  W = -Tm diag(beta e^gamma) K,
//
// and W and Tb do not depend on the state, so gdn_tri_kernel forms them for
// every chunk in parallel.  The sequential pass is then two products per chunk,
// U from S and S_{r+1} = e^{gamma_C} S_r + U^T diag(e^{gamma_C - gamma}) K, where
// the form without W has four dependent ones (K S^T, its sum over the waves
// that share a value tile, Tm R and the update).  Measured against that form
// (gdn_state_dma_kernel), dk = dv = 256: 521 -> 342 us at T = 20480 with 8 heads,
// 139 -> 104 us at T = 4096 with 32, for 10 us more in gdn_tri_kernel.
//
// What bounds the pass is the chain of chunks: there are only B H dv / 16 value
// tiles of S, two per compute unit at the 1.3B training shape and half of one
// for a long sequence of few heads, and a chunk must finish before the next one
// begins.  So one wave carries a value tile whole (16 columns of S^T, all key
// features, in accumulators: 64 registers at dk = 256), with no partial sums to
// exchange, and does nothing else: four more waves of the workgroup stream the
// chunk's W, Tb and K into LDS (global_load_lds, no registers), one its V slice
// and coefficients, and one brings the lines of later chunks into the XCD's L2.
#include "ccq_device.h"
#include "ccq_kernels.h"

namespace ccq {

// NPR value tiles (consumer waves) per workgroup.  LDS: two slots each of W | Tb,
// of K and of V slice | coefficients, refilled for the chunk after next as soon
// as they are free.
template <int DK, int NPR>
struct WyTile {
  static constexpr int C = kChunk, NLW = 4, BVS = 16 * NPR, NKH = DK / 32;
  static constexpr int NW = NPR + NLW + 2;  // consumers, loaders of W and K, the V loader, the prefetching wave
  static constexpr int WB = C * DK * 2, TB = 6 * 1024, VB = C * BVS * 2, FB = 2 * C * 4, KB = C * DK * 2;
  static constexpr int SW = WB + TB, SV = VB + FB;  // bytes of a W slot and of a V slot
  static constexpr int LDS = 2 * (SW + KB + SV) + 256;  // 256: where the prefetching wave's loads land
  // loads (of 1 KB) per loader wave of a W slot and a K slot, of the V loader of a V slot
  static constexpr int NWL = WB / 1024 / NLW + 2, NKL = KB / 1024 / NLW, NVL = VB / 1024 + 1;
};

// (At least eight waves per workgroup, padding the bound where there are fewer,
// keep the kernel within 256 registers, where the compiler leaves the
// accumulators in ordinary registers; given more, it moves them to and from the
// accumulation file around every scaling, 160 more instructions per chunk.)
template <int DK, int NPR>
__global__ __launch_bounds__(64 * (NPR + 6 < 8 ? 8 : NPR + 6)) void gdn_wy_state_kernel(const GdnArgs a) {
  typedef bf16_t T;
  typedef __attribute__((address_space(3))) void lds_void;
  typedef WyTile<DK, NPR> L;
  constexpr int C = kChunk, BVS = L::BVS, NKH = L::NKH, NCT = DK / 16, RB = DK * 2;
  static_assert(DK == 128 || DK == 256, "K rows of at least 16 pieces");
  static_assert(L::LDS <= 160 * 1024 && L::WB / 1024 % L::NLW == 0 && 2 * L::NKL + L::NWL < 64, "LDS and load counts");
  __shared__ __align__(1024) char smem[L::LDS];
  char* const sW = smem;
  char* const sK = smem + 2 * L::SW;
  char* const sV = sK + 2 * L::KB;

  const int nvt = a.dv / BVS;
  const int N = (a.T + C - 1) / C;
  const int lb = xcd_logical_block(blockIdx.x, gridDim.x);
  // heads in head-major order: the workgroups of consecutive logical blocks
  // (one compute-unit cluster) then hold one head of every sequence, which
  // balances the clusters when a packed batch's sequences differ in length
  const int hm = lb / nvt;
  const int bh = (hm % a.B) * a.H + hm / a.B;
  const int b = bh / a.H, h = bh % a.H;
  const Seq sq = seq_of(a.cu, b, a.T);
  const int NL = (sq.len + C - 1) / C;  // chunks walked (a packed sequence's own)
  const int l = lane_id(), g4 = l >> 4, c16 = l & 15;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int v0 = (lb % nvt) * BVS;
  const char* const wg = static_cast<const char*>(a.W) + (size_t)bh * N * L::WB;
  const char* const kg = static_cast<const char*>(a.k);
  const char* const tg = static_cast<const char*>(a.Tb) + (size_t)bh * N * kTbBytes;
  const char* const vg = static_cast<const char*>(a.v);
  const float* const fg = a.gam + (size_t)bh * N * 5 * C;

  if (w == NPR + L::NLW + 1) {
    // ---- prefetching wave ----
    // Brings the lines of the chunk kAhead ahead into this XCD's L2, each
    // workgroup of the head (they sit on one XCD) its share, one line per lane,
    // so that the loaders find them there: the time a slot has to be refilled is
    // shorter than a load from memory takes (one value tile per workgroup, T =
    // 20480: 442 us without it, 348 with).  The loaded words go to a corner of
    // LDS that nothing reads.
    constexpr int kAhead = 4;
    const int kl = a.H * DK * 2, vl = a.H * a.dv * 2, nvl = a.dv / 64;  // row pitches, lines per V row
    const int nline = (L::WB + L::KB + L::TB) / 128 + 10 + C * nvl;
    auto touch = [&](int ci) {
      const int nrow = min(C, sq.len - ci * C);
      const char* kc = kg + seq_off(sq, ci * C, h, a.H, DK) * 2;
      const char* vc = vg + seq_off(sq, ci * C, h, a.H, a.dv) * 2;
      for (int i = (lb % nvt) * 64 + l; i < nline; i += nvt * 64) {
        int x = i;
        const char* p;
        if (x < L::WB / 128) {
          p = wg + (size_t)ci * L::WB + 128 * x;
        } else if ((x -= L::WB / 128) < L::KB / 128) {
          p = kc + (size_t)min(x / (DK / 64), nrow - 1) * kl + 128 * (x % (DK / 64));
        } else if ((x -= L::KB / 128) < L::TB / 128) {
          p = tg + (size_t)ci * kTbBytes + 128 * x;
        } else if ((x -= L::TB / 128) < 10) {  // the chunk's decay coefficients
          p = reinterpret_cast<const char*>(fg + (size_t)ci * 5 * C) + 128 * x;
        } else {
          x -= 10;
          p = vc + (size_t)min(x / nvl, nrow - 1) * vl + 128 * (x % nvl);
        }
        __builtin_amdgcn_global_load_lds((const void*)p, (lds_void*)(smem + L::LDS - 256), 4, 0, 0);
      }
    };
    for (int ci = 2; ci < kAhead && ci < NL; ++ci) touch(ci);
#pragma unroll 1
    for (int ci = 0; ci < NL; ++ci) {
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_s_barrier();
      if (ci + kAhead < NL) touch(ci + kAhead);
    }
    wait_vm<0>();
    return;
  }

#define CCQ_LDS(src, dst, off) __builtin_amdgcn_global_load_lds((const void*)(src), (lds_void*)(dst), 16, off, 0)
  if (w == NPR + L::NLW) {
    // ---- V loader ----
    // The V rows of one head are H dv apart, on few of the L2's channels, and come
    // later than the contiguous operands: a wave of its own, since loads of one
    // wave return in order.
    constexpr int CPV = BVS / 8;  // 16-byte pieces per V row
    auto issue_v = [&](int ci) {
      char* sb = sV + (ci & 1) * L::SV;
      const int nrow = min(C, sq.len - ci * C);
      const char* vc = vg + (seq_off(sq, ci * C, h, a.H, a.dv) + v0) * 2;
#pragma unroll
      for (int it = 0; it < L::VB / 1024; ++it) {  // rows past the end repeat the last one
        const int row = it * (64 / CPV) + l / CPV;
        CCQ_LDS(vc + (uint32_t)min(row, nrow - 1) * (uint32_t)(a.H * a.dv * 2) + 16 * (l % CPV), sb + it * 1024, 0);
      }
      // e^{gamma_C - gamma_j} (row ddrow) and e^{gamma_C} (row 4): 512 bytes
      const float* cf = fg + ((size_t)ci * 5 + (l < 16 ? 3 : 4)) * C + 4 * (l & 15);
      if (l < 32) CCQ_LDS(cf, sb + L::VB, 0);
    };
    if (NL > 0) issue_v(0);
    if (NL > 1) issue_v(1);
#pragma unroll 1
    for (int ci = 0; ci < NL; ++ci) {
      if (ci + 1 < NL) wait_vm<L::NVL>();  // V(ci + 1) may be in flight
      else wait_vm<0>();
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_s_barrier();  // (the consumers have read the slot by now)
      if (ci + 2 < NL) issue_v(ci + 2);
    }
    return;
  }
  if (w >= NPR) {
    // ---- loaders of W and K ----
    // Per load: a uniform base, a lane offset and the LDS base (an immediate
    // offset moves both addresses).
    const int lw = w - NPR;
    const uint32_t lo16 = 16 * l;
    auto issue_w = [&](int ci) {
      char* sb = sW + (ci & 1) * L::SW;
      const char* wc = wg + (size_t)ci * L::WB;
#pragma unroll
      for (int it = 0; it < L::WB / 4096 / L::NLW; ++it) {  // 4 KB by each loader in turn
        const int o = (L::NLW * it + lw) * 4096;
        CCQ_LDS(wc + o + lo16, sb + o, 0);
        CCQ_LDS(wc + o + lo16, sb + o, 1024);
        CCQ_LDS(wc + o + lo16, sb + o, 2048);
        CCQ_LDS(wc + o + lo16, sb + o, 3072);
      }
      // Tb, one piece by each loader in turn (two of them twice, so that every
      // loader issues the same number)
#pragma unroll
      for (int it = 0; it < 2; ++it) {
        const int o = ((L::NLW * it + lw) % 6) * 1024;
        CCQ_LDS(tg + (size_t)ci * kTbBytes + o + lo16, sb + L::WB + o, 0);
      }
    };
    // K rows, whole chunks with offsets formed once; rows past the end repeat
    // the last one
    constexpr int CPK = DK / 8;  // 16-byte pieces per row
    uint32_t koff[L::NKL];
    auto row_offsets = [&](int nrow) {
#pragma unroll
      for (int it = 0; it < L::NKL; ++it) {
        const int row = (L::NLW * it + lw) * (64 / CPK) + l / CPK;
        koff[it] = (uint32_t)min(row, nrow - 1) * (uint32_t)(a.H * DK * 2) + 16 * ((l % CPK) ^ kswz(row));
      }
    };
    row_offsets(min(C, sq.len));
    auto issue_k = [&](int ci) {
      char* sb = sK + (ci & 1) * L::KB;
      if (ci > 0 && ci * C + C > sq.len) row_offsets(sq.len - ci * C);  // the last chunk, cut
      const char* kc = kg + seq_off(sq, ci * C, h, a.H, DK) * 2;
#pragma unroll
      for (int it = 0; it < L::NKL; ++it) CCQ_LDS(kc + koff[it], sb + (L::NLW * it + lw) * 1024, 0);
    };
    // Barriers of a chunk: (1) its W and V slots have landed and the K slot of
    // the chunk before is free; (2) its K slot has landed, its W and V slots are
    // free.  Loads return in order: what
    // was issued after the awaited slot may stay in flight (the K slot of the
    // same chunk or the W slot of the next, and the slot refilled last).
#pragma unroll 1
    for (int ci = 0; ci < 2 && ci < NL; ++ci) {
      issue_w(ci);
      issue_k(ci);
    }
#pragma unroll 1
    for (int ci = 0; ci < NL; ++ci) {
      if (ci + 1 >= NL) wait_vm<0>();
      else if (ci == 0) wait_vm<2 * L::NKL + L::NWL>();  // K(0), W(1), K(1) may be in flight
      else wait_vm<L::NKL + L::NWL>();                   // K(ci), W(ci + 1)
      __builtin_amdgcn_s_barrier();
      if (ci >= 1 && ci + 1 < NL) issue_k(ci + 1);
      if (ci + 1 >= NL) wait_vm<0>();
      else wait_vm<L::NKL + L::NWL>();                   // W(ci + 1), K(ci + 1)
      __builtin_amdgcn_s_barrier();
      if (ci + 2 < NL) issue_w(ci + 2);
    }
    return;
  }

#undef CCQ_LDS
  // ---- consumer wave: value tile w of the workgroup's slice ----
  const int v = v0 + 16 * w + c16;
  // S^T[c][v] in pair order: c = pair_feat(tc, g4) + r, so that the packed
  // operand of tiles 2m, 2m + 1 holds 8 consecutive features per lane group
  f32x4 S[NCT];
#pragma unroll
  for (int tc = 0; tc < NCT; ++tc) S[tc] = zero4();
  if (a.S0) {
    const float* s0 = a.S0 + ((size_t)bh * a.dv + v) * DK + 8 * g4;
#pragma unroll
    for (int tc = 0; tc < NCT; ++tc) S[tc] = *reinterpret_cast<const f32x4*>(s0 + pair_feat(tc, 0));
  }
  const int vt = (v0 >> 4) + w;
  T* st_base = static_cast<T*>(a.states) + ((size_t)vt * NKH * 16 + c16) * 32 + 8 * g4;
  T* u_base = static_cast<T*>(a.U) + ((size_t)vt * 2 * 16 + c16) * 32 + 8 * g4;
  typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;
  auto ldf = [](const char* p) {
    Frag<T> f;
    f.v = *reinterpret_cast<const bf16x8*>(p);
    return f;
  };
  auto tr2 = [](const char* p, int off) {  // two transposing reads, the second `off` bytes on
    const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)p);
    const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(p + off));
    Frag<T> f;
    f.v = bf16x8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return f;
  };
  // transposing reads of K, rows 4 g4 + j / 4 (j = c16), piece 4 m + j % 4
  // (permuted), half t % 2: the permutation touches the low four bits of the
  // piece index only, so block m differs from block m % 4 by a constant
  int koff[4];
  {
    const int j = c16, rr = 4 * g4 + (j >> 2), rs = kswz(rr);
#pragma unroll
    for (int q = 0; q < 4; ++q) koff[q] = rr * RB + 16 * ((4 * q + (j & 3)) ^ rs);
  }

  int until = 0;  // chunks until the next stored state
#pragma unroll 1
  for (int ci = 0; ci < NL; ++ci) {
    const char* wb = sW + (ci & 1) * L::SW;
    const char* kb = sK + (ci & 1) * L::KB;
    const char* vb = sV + (ci & 1) * L::SV;
    Frag<T> sf[NKH];
#pragma unroll
    for (int m = 0; m < NKH; ++m) sf[m] = acc_pair_frag<T>(S[2 * m], S[2 * m + 1]);
    lds_barrier();  // this chunk's W and V slots have landed
    // U = Tb V + W S^T, token tiles I in accumulators
    const float* Fb = reinterpret_cast<const float*>(vb + L::VB);
    const float eC = Fb[C];
    f32x4 U[4];
#pragma unroll
    for (int I = 0; I < 4; ++I) U[I] = zero4();
    {
      const char* pv = vb + (4 * g4 + (c16 >> 2)) * (2 * BVS) + 32 * w + 8 * (c16 & 3);
      const Frag<T> vf0 = tr2(pv, 16 * 2 * BVS), vf1 = tr2(pv + 32 * 2 * BVS, 16 * 2 * BVS);
      const char* tb = wb + L::WB + 16 * l;  // blocks (0, 0), (1, 0), (2, 0), (2, 1), (3, 0), (3, 1)
      mma(U[0], ldf(tb), vf0);
      mma(U[1], ldf(tb + 1024), vf0);
      mma(U[2], ldf(tb + 2048), vf0);
      mma(U[3], ldf(tb + 4096), vf0);
      mma(U[2], ldf(tb + 3072), vf1);
      mma(U[3], ldf(tb + 5120), vf1);
    }
#pragma unroll
    for (int m = 0; m < NKH; ++m) {
#pragma unroll
      for (int I = 0; I < 4; ++I) mma(U[I], ldf(wb + (I * NKH + m) * 1024 + 16 * l), sf[m]);
      S[2 * m] *= eC;
      S[2 * m + 1] *= eC;
    }
    Frag<T> uf[2], ud[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) uf[q] = acc_pair_frag<T>(U[2 * q], U[2 * q + 1]);
#pragma unroll
    for (int I = 0; I < 4; ++I) U[I] *= *reinterpret_cast<const f32x4*>(Fb + 16 * I + 4 * g4);
#pragma unroll
    for (int q = 0; q < 2; ++q) ud[q] = acc_pair_frag<T>(U[2 * q], U[2 * q + 1]);
    lds_barrier();  // this chunk's K slot has landed, its W and V slots are free
    // S^T <- e^{gamma_C} S^T + K^T diag(e^{gamma_C - gamma}) U
#pragma unroll
    for (int tc = 0; tc < NCT; ++tc) {
      const int m = tc >> 1;
      const char* pk = kb + koff[m & 3] + (m >> 2) * 256 + 8 * (tc & 1);
#pragma unroll
      for (int kq = 0; kq < 2; ++kq) mma(S[tc], tr2(pk + 32 * kq * RB, 16 * RB), ud[kq]);
    }
    // S_r (every sstride-th chunk) and U^T, fragment-native
    if (until == 0) {
      T* st_out = st_base + ((size_t)bh * N + ci) * a.dv * DK;
#pragma unroll
      for (int m = 0; m < NKH; ++m) store_frag(st_out + 16 * 32 * m, sf[m]);
      until = a.sstride;
    }
    --until;
    T* u_out = u_base + ((size_t)bh * N + ci) * a.dv * C;
    store_frag(u_out, uf[0]);
    store_frag(u_out + 16 * 32, uf[1]);
  }

  if (a.ST) {
    float* st = a.ST + ((size_t)bh * a.dv + v) * DK + 8 * g4;
#pragma unroll
    for (int tc = 0; tc < NCT; ++tc) *reinterpret_cast<f32x4*>(st + pair_feat(tc, 0)) = S[tc];
  }
}

namespace {
template <int DK, int NPR>
hipError_t run_wy(const GdnArgs& a, hipStream_t st) {
  const int nblk = a.B * a.H * (a.dv / (16 * NPR));
  if (nblk == 0) return hipSuccess;
  hipLaunchKernelGGL((gdn_wy_state_kernel<DK, NPR>), dim3(nblk), dim3(64 * WyTile<DK, NPR>::NW), 0, st, a);
  return hipGetLastError();
}
// One value tile per workgroup while every tile can have a compute unit of its
// own, else two; at dk = 128, four where two would take a second round.
template <int DK>
hipError_t run_wy_dk(const GdnArgs& a, hipStream_t st) {
  const long long slices = (long long)a.B * a.H * (a.dv / 16);
  if (slices <= 256) return run_wy<DK, 1>(a, st);
  if constexpr (DK == 128)
    if (slices > 512) return run_wy<DK, 4>(a, st);
  return run_wy<DK, 2>(a, st);
}
}  // namespace

// Where the WY form is used (us per call on one card, WY against the other form,
// B x H x dk x dv).  Forming W costs gdn_tri_kernel 10 us at 2048 chunk-heads of
// dk = 256, so short sequences keep the other form: dk = 256 from 8 chunks with
// one value tile per compute unit (1 x 8 x 256 x 256, T = 256: 55.4 against 54.7,
// T = 512: 63.1 against 65.2, T = 4096: 185 against 213) and from 16 with more
// (4 x 8 x 256 x 256, T = 512: 88.5 against 87.1, T = 2048: 205 against 210, T =
// 4096: 325 against 337); dk = 128 from 4 (1 x 4 x 128 x 128, T = 128: 34.9 against
// 33.7, T = 256: 35.9 against 37.6; 8 x 4 x 128 x 256, T = 4096: 213 against 242).
// A training step stores every S_r, which the few consumer waves issue behind
// the loaders: up to one value tile of 256 features per compute unit (training
// step 1 x 8 x 256 x 256, T = 2048: 405 against 418; 8 x 4 x 128 x 256: 494
// against 497; 4 x 8 x 256 x 256: 907 against 890).
bool gdn_wy(long long bh, long long nc, int dk, int dv, bool is_bf16, bool every_state) {
  if (!is_bf16 || (dk != 128 && dk != 256)) return false;
  const long long tiles = bh * (dv / 16);
  if (every_state && tiles * dk > 65536) return false;
  return nc >= (dk == 128 ? 4 : tiles <= 256 ? 8 : 16);
}

hipError_t launch_gdn_wy_state(const GdnArgs& a, hipStream_t st) {
  if (!a.W || !a.Tb) return hipErrorInvalidValue;
  switch (a.dk) {
    case 128: return run_wy_dk<128>(a, st);
    case 256: return run_wy_dk<256>(a, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace ccq
