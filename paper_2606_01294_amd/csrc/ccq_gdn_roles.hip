// ccq_gdn_roles.hip -- Gated DeltaNet state pass with the waves in roles (bf16,
// dk = 128 and 256).
//
// The recurrence of gdn_state_kernel (ccq_gdn.hip), for each chunk
//
//   R = diag(beta) (V - diag(e^gamma) K S_r^T),  U = Tm R,
//   S_{r+1} = e^{gamma_C} S_r + U^T diag(e^{gamma_C - gamma}) K.
//
// What bounds the pass is the chain of chunks: there are only B H dv / 16 value
// tiles of S, two per compute unit at the 1.3B training shape and half of one
// for a long sequence of few heads, and a chunk must finish before the next one
// begins.  So one wave carries a value tile whole (16 columns of S^T, all key
// features, in accumulators: 64 registers at dk = 256), with no partial sums to
// exchange through LDS, and does nothing else: four more waves of the workgroup
// stream the operands of the next two chunks into a ring of three LDS slots
// (global_load_lds, no registers).  One barrier a chunk.
//
// Measured against the form it took the place of (the features of a tile split
// over four waves that exchange partial sums through LDS), same bits: 521 -> 390
// us at T = 20480 with 8 heads (dk = dv = 256), 139 -> 102 us at T = 4096 with
// 32, 60 -> 40 us on 8 packed sequences of up to 2048 tokens x 4 heads (dk = 128,
// dv = 256), 152 -> 145 us in a training step at T = 4096 (every state stored).
// It is no slower from one chunk on (whole forwards of 1 to 32 chunks, 32 to 1024
// value tiles: 1.00 to 1.5 times as fast; training steps 1.00 to 1.08), so every
// call of these types takes it.  A chunk takes the wave about 2900 cycles, 1200 of
// them products.
//
// (The products without V could be formed ahead of the pass: U = Tb V + W S_r^T
// with Tb = Tm diag(beta), W = -Tm diag(beta e^gamma) K leaves two products in
// the chain and took 342 us at T = 20480.  It is not used: W rounded to bf16
// and the cancellation of the two terms after it put S_T 1.3 to 1.4 times as far
// from the exact result where the state predicts the values.)
#include "ccq_device.h"
#include "ccq_kernels.h"

namespace ccq {

// NPR value tiles (consumer waves) per workgroup.  A slot: K | Tm | V slice |
// coefficients, unpadded, K and Tm with their 16-byte pieces permuted per row
// (kswz, tswz).
template <int DK, int NPR>
struct RolesTile {
  static constexpr int C = kChunk, NLW = 4, BVS = 16 * NPR, NKH = DK / 32;
  static constexpr int NW = NPR + NLW;  // consumers, loaders
  static constexpr int KB = C * DK * 2, TB = C * C * 2, VB = C * BVS * 2, FB = 4 * C * 4;
  static constexpr int SB = KB + TB + VB + FB, NSLOT = 3, LDS = NSLOT * SB;
  // loads (of 1 KB) per loader wave and chunk
  static constexpr int NKL = KB / 1024 / NLW, NTL = TB / 1024 / NLW, NV = VB / 1024, NVL = (NV + NLW - 1) / NLW;
  static constexpr int NL = NKL + NTL + NVL + 1;
};

// NG: the key features are summed in NG groups.
// (At least eight waves per workgroup, padding the bound where there are fewer,
// keep the kernel within 256 registers, where the compiler leaves the
// accumulators in ordinary registers; given more, it moves them to and from the
// accumulation file around every scaling.)
template <int DK, int NPR, int NG>
__global__ __launch_bounds__(64 * (NPR + 4 < 8 ? 8 : NPR + 4)) void gdn_state_roles_kernel(const GdnArgs a) {
  typedef bf16_t T;
  typedef __attribute__((address_space(3))) void lds_void;
  typedef RolesTile<DK, NPR> L;
  constexpr int C = kChunk, BVS = L::BVS, NKH = L::NKH, NCT = DK / 16, RB = DK * 2;
  static_assert(DK == 128 || DK == 256, "K rows of at least 16 pieces");
  static_assert(L::LDS <= 160 * 1024 && L::NKL >= 1 && L::KB / 1024 % L::NLW == 0 && L::TB / 1024 % L::NLW == 0 &&
                    (L::NV % L::NLW == 0 || L::NLW % L::NV == 0) && 2 * L::NL < 64,
                "LDS and load counts");
  static_assert(NKH % NG == 0, "feature groups");
  __shared__ __align__(1024) char smem[L::LDS];

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
  const int NLC = (sq.len + C - 1) / C;  // chunks walked (a packed sequence's own)
  const int l = lane_id(), g4 = l >> 4, c16 = l & 15;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int v0 = (lb % nvt) * BVS;

  if (w >= NPR) {
    // ---- loaders ----
    // Each issues the same number of loads per chunk (a piece that not every
    // wave can have is shared out by lanes: lane i of a piece lands at its base
    // + 16 i whichever lanes are active).  Row offsets are formed once for whole
    // chunks; rows past the end of the sequence read the last row (finite data;
    // the chunk transform zeroes their contribution).
#define CCQ_LDS(src, dst) __builtin_amdgcn_global_load_lds((const void*)(src), (lds_void*)(dst), 16, 0, 0)
    const int lw = w - NPR;
    const char* const kg = static_cast<const char*>(a.k);
    const char* const vg = static_cast<const char*>(a.v);
    const char* const tg = static_cast<const char*>(a.Tm) + (size_t)bh * N * L::TB;
    const float* const fg = a.gam + (size_t)bh * N * 5 * C;
    constexpr int CPK = DK / 8, CPV = BVS / 8;  // 16-byte pieces per row
    constexpr int SH = L::NV >= L::NLW ? 1 : L::NLW / L::NV, LPW = 64 / SH;  // loaders sharing a V piece
    uint32_t koff[L::NKL], voff[L::NVL], toff[L::NTL];
    auto row_offsets = [&](int nrow) {
#pragma unroll
      for (int it = 0; it < L::NKL; ++it) {
        const int row = (L::NLW * it + lw) * (64 / CPK) + l / CPK;
        koff[it] = (uint32_t)min(row, nrow - 1) * (uint32_t)(a.H * RB) + 16 * ((l % CPK) ^ kswz(row));
      }
#pragma unroll
      for (int it = 0; it < L::NVL; ++it) {
        const int row = (SH == 1 ? L::NLW * it + lw : lw / SH) * (64 / CPV) + l / CPV;
        voff[it] = (uint32_t)min(row, nrow - 1) * (uint32_t)(a.H * a.dv * 2) + 16 * (l % CPV);
      }
    };
#pragma unroll
    for (int it = 0; it < L::NTL; ++it) {
      const int row = (L::NLW * it + lw) * 8 + l / 8;
      toff[it] = row * (C * 2) + 16 * ((l % 8) ^ tswz(row));
    }
    row_offsets(min(C, sq.len));
    auto issue = [&](int ci) {
      char* sb = smem + (ci % L::NSLOT) * L::SB;
      if (ci > 0 && ci * C + C > sq.len) row_offsets(sq.len - ci * C);  // the last chunk, cut
      const char* kc = kg + seq_off(sq, ci * C, h, a.H, DK) * 2;
      const char* vc = vg + (seq_off(sq, ci * C, h, a.H, a.dv) + v0) * 2;
#pragma unroll
      for (int it = 0; it < L::NVL; ++it)
        if (SH == 1 || l / LPW == lw % SH)
          CCQ_LDS(vc + voff[it], sb + L::KB + L::TB + (SH == 1 ? L::NLW * it + lw : lw / SH) * 1024);
#pragma unroll
      for (int it = 0; it < L::NKL; ++it) CCQ_LDS(kc + koff[it], sb + (L::NLW * it + lw) * 1024);
#pragma unroll
      for (int it = 0; it < L::NTL; ++it)
        CCQ_LDS(tg + (size_t)ci * L::TB + toff[it], sb + L::KB + (L::NLW * it + lw) * 1024);
      // coefficient rows 1..4: beta e^gamma, beta, e^{gamma_C - gamma}, e^{gamma_C}
      if (l / (64 / L::NLW) == lw) CCQ_LDS(fg + ((size_t)ci * 5 + 1) * C + 4 * l, sb + L::KB + L::TB + L::VB);
    };
    if (NLC > 0) issue(0);
    if (NLC > 1) issue(1);
    // At the barrier of chunk ci its slot has landed (loads return in order: the
    // next chunk's may stay in flight) and the consumers have read the slot of
    // chunk ci - 1, which chunk ci + 2 then takes.
#pragma unroll 1
    for (int ci = 0; ci < NLC; ++ci) {
      if (ci + 1 < NLC) wait_vm<L::NL>();
      else wait_vm<0>();
      __builtin_amdgcn_s_barrier();
      if (ci + 2 < NLC) issue(ci + 2);
    }
    return;
#undef CCQ_LDS
  }

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
  auto tr = [](const char* p) { return __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)p); };
  // The permutation of K touches the low four bits of the piece index only, so a
  // lane's block m of 32 features lies 256 (m / 4) bytes on from block m % 4.
  // krow: row c16, piece 4 m + g4 (row operands); kcol: transposing reads, rows
  // 4 g4 + j / 4 (j = c16), piece 4 m + j % 4 (+ 8 bytes for odd tiles)
  int krow[4], kcol[4];
  {
    const int rr = 4 * g4 + (c16 >> 2);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      krow[q] = c16 * RB + 16 * ((4 * q + g4) ^ kswz(c16));
      kcol[q] = rr * RB + 16 * ((4 * q + (c16 & 3)) ^ kswz(rr));
    }
  }
  const int trow = c16 * (C * 2) + 16 * (g4 ^ tswz(c16));  // Tm row c16, columns 8 g4 ..; 32 on: ^ 64
  const int vrow = (4 * g4 + (c16 >> 2)) * (2 * BVS) + 32 * w + 8 * (c16 & 3);

  int until = 0;  // chunks until the next stored state
#pragma unroll 1
  for (int ci = 0; ci < NLC; ++ci) {
    const char* kb = smem + (ci % L::NSLOT) * L::SB;
    const char* tb = kb + L::KB;
    const char* vb = tb + L::TB;
    const float* Fb = reinterpret_cast<const float*>(vb + L::VB);
    Frag<T> sf[NKH];
#pragma unroll
    for (int m = 0; m < NKH; ++m) sf[m] = acc_pair_frag<T>(S[2 * m], S[2 * m + 1]);
    lds_barrier();  // this chunk's slot has landed, the one before is free
    // LDS reads run one step of products ahead of their use (the scheduling
    // barriers keep the compiler from sinking them to it): the wave is alone on
    // its SIMD's matrix core, so nothing else hides them.
    // R = beta V - beta e^gamma K S_r^T: token tile J in accumulators, the
    // feature groups' sums added in order
    Frag<T> kf[2][NKH], tm[4][2];
    auto read_k = [&](int J) {
#pragma unroll
      for (int m = 0; m < NKH; ++m) kf[J & 1][m] = ldf(kb + krow[m & 3] + (m >> 2) * 256 + 16 * J * RB);
    };
    const float eC = Fb[3 * C];
    read_k(0);
    f32x4 R[4];
#pragma unroll
    for (int J = 0; J < 4; ++J) {
      const bf16x4 vv = tr(vb + vrow + 16 * J * 2 * BVS);
      const f32x4 bg = *reinterpret_cast<const f32x4*>(Fb + 16 * J + 4 * g4);
      const f32x4 bj = *reinterpret_cast<const f32x4*>(Fb + C + 16 * J + 4 * g4);
      if (J < 3) {
        read_k(J + 1);
      } else {  // Tm (rows stored in acc_pos order)
#pragma unroll
        for (int I = 0; I < 4; ++I) {
          tm[I][0] = ldf(tb + trow + 16 * I * (C * 2));
          tm[I][1] = ldf(tb + (trow ^ 64) + 16 * I * (C * 2));
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      f32x4 x[NG];
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        x[g] = zero4();
#pragma unroll
        for (int mm = 0; mm < NKH / NG; ++mm) mma(x[g], kf[J & 1][g * (NKH / NG) + mm], sf[g * (NKH / NG) + mm]);
      }
#pragma unroll
      for (int t = 0; t < NCT / 4; ++t) S[NCT / 4 * J + t] *= eC;
      f32x4 sum = x[0];
#pragma unroll
      for (int g = 1; g < NG; ++g) sum += x[g];
#pragma unroll
      for (int r = 0; r < 4; ++r) R[J][r] = bj[r] * f32(vv[r]) - bg[r] * sum[r];
    }
    const Frag<T> rf0 = acc_pair_frag<T>(R[0], R[1]), rf1 = acc_pair_frag<T>(R[2], R[3]);
    // K^T of TB feature tiles at a time, for the update
    constexpr int TB = 4;
    Frag<T> tf[2][TB][2];
    auto read_t = [&](int tc0, Frag<T>(&f)[TB][2]) {
#pragma unroll
      for (int t = 0; t < TB; ++t) {
        const int tc = tc0 + t, m = tc >> 1;
        const char* pk = kb + kcol[m & 3] + (m >> 2) * 256 + 8 * (tc & 1);
#pragma unroll
        for (int kq = 0; kq < 2; ++kq) {
          const bf16x4 lo = tr(pk + 32 * kq * RB), hi = tr(pk + (32 * kq + 16) * RB);
          f[t][kq].v = bf16x8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        }
      }
    };
    f32x4 dd[4];
#pragma unroll
    for (int I = 0; I < 4; ++I) dd[I] = *reinterpret_cast<const f32x4*>(Fb + 2 * C + 16 * I + 4 * g4);
    read_t(0, tf[0]);
    __builtin_amdgcn_sched_barrier(0);
    // U = Tm R
    f32x4 U[4];
#pragma unroll
    for (int I = 0; I < 4; ++I) {
      U[I] = zero4();
      mma(U[I], tm[I][0], rf0);
    }
#pragma unroll
    for (int I = 0; I < 4; ++I) mma(U[I], tm[I][1], rf1);
    Frag<T> uf[2], ud[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      uf[q] = acc_pair_frag<T>(U[2 * q], U[2 * q + 1]);
      U[2 * q] *= dd[2 * q];
      U[2 * q + 1] *= dd[2 * q + 1];
      ud[q] = acc_pair_frag<T>(U[2 * q], U[2 * q + 1]);
    }
    // S^T <- e^{gamma_C} S^T + K^T diag(e^{gamma_C - gamma}) U
#pragma unroll
    for (int tb4 = 0; tb4 < NCT / TB; ++tb4) {
      if (tb4 + 1 < NCT / TB) read_t(TB * (tb4 + 1), tf[(tb4 + 1) & 1]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int kq = 0; kq < 2; ++kq)
#pragma unroll
        for (int t = 0; t < TB; ++t) mma(S[TB * tb4 + t], tf[tb4 & 1][t][kq], ud[kq]);
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
template <int DK, int NPR, int NG = 4>
hipError_t run_roles(const GdnArgs& a, hipStream_t st) {
  const int nblk = a.B * a.H * (a.dv / (16 * NPR));
  if (nblk == 0) return hipSuccess;
  hipLaunchKernelGGL((gdn_state_roles_kernel<DK, NPR, NG>), dim3(nblk), dim3(64 * RolesTile<DK, NPR>::NW), 0, st, a);
  return hipGetLastError();
}
// One value tile per workgroup while every tile can have a compute unit of its
// own, else two; at dk = 128, four where two would take a second round.  (The
// features' sum keeps the order it has had at each of these shapes: from 1024
// tiles of dk = 128 on, two groups.)
template <int DK>
hipError_t run_roles_dk(const GdnArgs& a, hipStream_t st) {
  const long long slices = (long long)a.B * a.H * (a.dv / 16);
  if (slices <= 256) return run_roles<DK, 1>(a, st);
  if constexpr (DK == 128) {
    if (slices >= 1024) return run_roles<DK, 4, 2>(a, st);
    if (slices > 512) return run_roles<DK, 4>(a, st);
  }
  return run_roles<DK, 2>(a, st);
}
}  // namespace

hipError_t launch_gdn_state_roles(const GdnArgs& a, hipStream_t st) {
  switch (a.dk) {
    case 128: return run_roles_dk<128>(a, st);
    case 256: return run_roles_dk<256>(a, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace ccq
