// The L = 4 edge pass through per-edge matrices (cp_edge_mat_impl.hpp): when it
// is taken, its factor operands and its dispatch.
#include "cp_edge_mat_impl.hpp"

namespace tdn {
namespace mat_detail {

#define TDN_MAT(RS, NT, BF, ATT, FG) \
  extern template hipError_t launch_mat<RS, NT, BF, ATT, FG>(const EdgeArgs&, hipStream_t);
#define TDN_MAT_RS(RS)               \
  TDN_MAT(RS, 3, false, false, false) \
  TDN_MAT(RS, 4, false, false, false) \
  TDN_MAT(RS, 3, false, true, false)  \
  TDN_MAT(RS, 4, false, true, false)  \
  TDN_MAT(RS, 3, false, false, true)  \
  TDN_MAT(RS, 4, false, false, true)  \
  TDN_MAT(RS, 4, true, false, false)  \
  TDN_MAT(RS, 8, true, false, false)
TDN_MAT_RS(6)
TDN_MAT_RS(8)
#undef TDN_MAT_RS
#undef TDN_MAT

namespace {

// The builder's factor operands, per rank step s of 16 and lane (h, l): EF
// 2^-e_E, row l, ranks 16 s + 8 h + j in fp32 ([RS][2][64 lanes] x 16 bytes);
// KF 2^-e_K, row l and the same ranks in two fp16 parts ([RS][2][64 lanes] x
// 16 bytes); then MatConst.  Zero past d and R.  One wave per step, every
// workgroup taking the factors' largest magnitudes itself; the last workgroup
// writes MatConst.
__global__ __launch_bounds__(256) void k_mat_factor(int R, int RS, int n_radial, const float* __restrict__ EF,
                                                    const float* __restrict__ KF, const float* __restrict__ B,
                                                    const float* __restrict__ Wrad, char* __restrict__ out) {
  __shared__ float red[16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  float mE = 0.f, mK = 0.f;
#pragma unroll 4
  for (int i = tid; i < kD * R; i += 256) {
    mE = fmaxf(mE, fabsf(EF[i]));
    mK = fmaxf(mK, fabsf(KF[i]));
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    mE = fmaxf(mE, __shfl_xor(mE, o));
    mK = fmaxf(mK, __shfl_xor(mK, o));
  }
  if (lane == 0) {
    red[wave] = mE;
    red[4 + wave] = mK;
  }
  __syncthreads();
  const int eE = f16_split_exponent(fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3])));
  const int eK = f16_split_exponent(fmaxf(fmaxf(red[4], red[5]), fmaxf(red[6], red[7])));
  const float sE = ldexpf(1.f, -eE), sK = ldexpf(1.f, -eK);
  if (blockIdx.x == gridDim.x - 1) {
    // the largest row norms of the scaled factors, a row per wave; the largest
    // of 5 |B_r| max_q |Wrad[q, r]| over the ranks
    float nE = 0.f, nK = 0.f, gb = 0.f;
    for (int k = wave; k < kD; k += 4) {
      float e = 0.f, f = 0.f;
      for (int r = lane; r < R; r += kWave) {
        const float u = EF[k * R + r] * sE, v = KF[k * R + r] * sK;
        e += u * u;
        f += v * v;
      }
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) {
        e += __shfl_xor(e, o);
        f += __shfl_xor(f, o);
      }
      nE = fmaxf(nE, e);
      nK = fmaxf(nK, f);
    }
    if (tid < R) {
      float n2 = 0.f, w = 0.f;
      for (int k = 0; k < kD; ++k) n2 += B[k * R + tid] * B[k * R + tid];
      for (int q = 0; q < n_radial; ++q) w = fmaxf(w, fabsf(Wrad[q * R + tid]));
      gb = 5.01f * sqrtf(n2) * w;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) gb = fmaxf(gb, __shfl_xor(gb, o));
    __syncthreads();
    if (lane == 0) {
      red[wave] = nE;
      red[4 + wave] = nK;
      red[8 + wave] = gb;
    }
    __syncthreads();
    if (tid == 0) {
      MatConst c;
      c.e_fac = eE + eK;
      int es = 0;
      (void)frexpf(sqrtf(fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]))) *
                       sqrtf(fmaxf(fmaxf(red[4], red[5]), fmaxf(red[6], red[7]))) * 1.01f, &es);
      c.e_split = es < 14 ? 0 : (es > 60 ? 46 : es - 14);
      c.g_bound = fmaxf(fmaxf(red[8], red[9]), fmaxf(red[10], red[11]));
      if (!(c.g_bound > 1e-30f) || !(c.g_bound < 1e30f)) c.g_bound = c.g_bound >= 1e30f ? 1e30f : 1e-30f;
      *reinterpret_cast<MatConst*>(out + RS * 4096) = c;
    }
    return;
  }
  const int s = blockIdx.x * 4 + wave;
  if (s >= RS) return;
  const int l = lane & 31, r0 = 16 * s + 8 * (lane >> 5);
  float e[8];
  uint32_t w[2][4];
#pragma unroll
  for (int j = 0; j < 8; j += 2) {
    float k[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int r = r0 + j + q;
      const bool ok = l < kD && r < R;
      e[j + q] = ok ? EF[l * R + r] * sE : 0.f;
      k[q] = ok ? KF[l * R + r] * sK : 0.f;
    }
    split_f16x2_pair(k[0], k[1], w[0][j / 2], w[1][j / 2]);
  }
  float4* eo = reinterpret_cast<float4*>(out) + 2 * s * kWave + lane;
  eo[0] = make_float4(e[0], e[1], e[2], e[3]);
  eo[kWave] = make_float4(e[4], e[5], e[6], e[7]);
  u32x4* ko = reinterpret_cast<u32x4*>(out + RS * 2048) + 2 * s * kWave + lane;
  ko[0] = u32x4{w[0][0], w[0][1], w[0][2], w[0][3]};
  ko[kWave] = u32x4{w[1][0], w[1][1], w[1][2], w[1][3]};
}

template <bool BF, bool ATT, bool FG>
hipError_t dispatch(const EdgeArgs& a, hipStream_t s) {
  const bool r3 = a.R <= 96;
  if constexpr (BF) {
    if (a.C <= 128) return r3 ? launch_mat<6, 4, true, false>(a, s) : launch_mat<8, 4, true, false>(a, s);
    return r3 ? launch_mat<6, 8, true, false>(a, s) : launch_mat<8, 8, true, false>(a, s);
  } else {
    // three or four tiles per applier, two groups of columns above 128
    const int n_ct = (a.C + kTile - 1) / kTile, groups = n_ct > 4 ? 2 : 1;
    if ((n_ct + groups - 1) / groups == 3)
      return r3 ? launch_mat<6, 3, false, ATT, FG>(a, s) : launch_mat<8, 3, false, ATT, FG>(a, s);
    return r3 ? launch_mat<6, 4, false, ATT, FG>(a, s) : launch_mat<8, 4, false, ATT, FG>(a, s);
  }
}

}  // namespace
}  // namespace mat_detail

// Both forms measured on batches of 50-atom molecules (2360 edges each), whole
// forward, us (rank form / this one):
//   fp32, 64 molecules: R, C = 128, 128: 463 / 382; 128, 48: 375 / 335; 128, 32:
//     322 / 319; 96, 96: 336 / 303; 96, 64: 256 / 360; 80, 80: 330 / 294; 128,
//     256: 930 / 766; 64, 128: 304 / 334
//   bf16, 64 molecules: 128, 128: 360 / 227; 128, 32: 305 / 207; 96, 128: 245 /
//     245; 72, 160: 321 / 243; 80, 80: 228 / 235; 64, 256: 314 / 303
//   fp32, R = C = 128: 8 molecules 98 / 109, 16: 153 / 173, 24: 209 / 167
// (the rank form steps at 32 and 64 ranks and 64 channels).  Below a range for
// every team of the device the teams' latency decides, and the rank form's
// waves have less of it.
bool mat_use(int L, int R, int C, bool bf16, int n_range) {
  if (L != 4 || R <= 64 || R > 128) return false;
  if (R > 96 ? C <= (bf16 ? 16 : 32) : C <= (bf16 ? 128 : 64)) return false;
  const int groups = !bf16 && C > 128 ? 2 : 1;
  return n_range * groups >= mat_detail::kTeams * device_cus();
}

hipError_t launch_cp_edge_mat(const EdgeArgs& a, hipStream_t s) {
  using namespace mat_detail;
  if (a.parts != 1 && a.parts != 2) return hipErrorInvalidValue;
  if (!mat_use(a.L, a.R, a.C, a.parts == 1, a.n_range) || a.n_range > a.E) return hipErrorInvalidValue;
  if (a.n_radial < 2 || a.n_radial > 16 || a.C > 256 || !a.ef_ops || (a.parts == 2 && !a.row_scale))
    return hipErrorInvalidValue;
  if (a.fa_global && (a.parts != 2 || a.alpha)) return hipErrorInvalidValue;
  if (a.alpha && (a.parts != 2 || a.n_heads < 1 || a.C % (kTile * a.n_heads) != 0)) return hipErrorInvalidValue;
  const int RS = 2 * ((a.R + kTile - 1) / kTile);
  if (size_t(RS) * 4096 + sizeof(MatConst) > edge_ef_bytes(a.d, a.R)) return hipErrorInvalidValue;
  k_mat_factor<<<dim3((RS + 3) / 4 + 1), dim3(256), 0, s>>>(a.R, RS, a.n_radial, a.EF, a.KF, a.Bf, a.radial_w,
                                                           static_cast<char*>(a.ef_ops));
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (a.parts == 1)
    e = dispatch<true, false, false>(a, s);
  else if (a.fa_global)
    e = dispatch<false, false, true>(a, s);
  else
    e = a.alpha ? dispatch<false, true, false>(a, s) : dispatch<false, false, false>(a, s);
  if (e != hipSuccess) return e;
  return launch_range_fixup(a, s);
}

}  // namespace tdn
