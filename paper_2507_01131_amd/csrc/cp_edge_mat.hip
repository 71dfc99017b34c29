// The L = 4 edge pass through per-edge matrices (cp_edge_mat_impl.hpp): when it
// is taken, its factor operands and its dispatch.
#include "cp_edge_mat_impl.hpp"

namespace tdn {
namespace mat_detail {

#define TDN_MAT(RS, NT, BF, ATT, FG) \
  extern template hipError_t launch_mat<RS, NT, BF, ATT, FG>(const EdgeArgs&, hipStream_t);
#define TDN_MAT_RS(RS)                \
  TDN_MAT(RS, 3, false, false, false) \
  TDN_MAT(RS, 4, false, false, false) \
  TDN_MAT(RS, 3, false, true, false)  \
  TDN_MAT(RS, 4, false, true, false)  \
  TDN_MAT(RS, 3, false, false, true)  \
  TDN_MAT(RS, 4, false, false, true)  \
  TDN_MAT(RS, 8, true, false, false)
TDN_MAT_RS(6)
TDN_MAT_RS(8)
TDN_MAT(8, 4, true, false, false)
#undef TDN_MAT_RS
#undef TDN_MAT

namespace {

// Exponent of a magnitude as frexp gives it; kNone for 0, and for an infinity or
// NaN (which stay in the operands and take no part in the scales).
constexpr int kNone = -(1 << 20);
__device__ __forceinline__ int mag_exp(float v) {
  int e = kNone;
  if (v != 0.f && fabsf(v) <= 3.4028234e38f) (void)frexpf(v, &e);
  return e;
}

// The builder's factor operands, per rank step s of 16 and lane (h, l): EF,
// row l, ranks 16 s + 8 h + j in fp32 ([RS][2][64 lanes] x 16 bytes); KF, row l
// and the same ranks in two fp16 parts ([RS][2][64 lanes] x 16 bytes), both
// scaled per row and then per column; zero past d and R (block 0).  Then the rest
// of MatOps (block 1).  Both blocks find the scales, with exponents as integers.
// Bound by the latency of its phases and, as a lone wave issues an instruction
// every eight cycles, by how many waves share them: 7 us; 12.5 with four waves a
// block and 15 with a step's operands per wave and the norms a row per wave (8.8
// with one scale per factor, in the latter form).
__global__ __launch_bounds__(1024) void k_mat_factor(int R, int RS, int n_radial, const float* __restrict__ EF,
                                                     const float* __restrict__ KF, const float* __restrict__ B,
                                                     const float* __restrict__ Wrad, char* __restrict__ out) {
  constexpr int kMost = 128, kParts = 8, kRowsPer = (kD + kParts - 1) / kParts;
  __shared__ float sF[2][kD][kMost + 1], sPart[kParts][kMost];
  __shared__ int sG[2][kMost], sCol[3][kMost], sRow[2][kTile], sTop[3], sMax[18];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int rank = tid & (kMost - 1), part = tid / kMost;  // rows part, part + 8, ... of a column each
  const int rc = min(rank, R - 1);
  const bool in = rank < R;
  // (all loads in flight at once)
  float v[2][kRowsPer], b[kRowsPer], w[2];
#pragma unroll
  for (int j = 0; j < kRowsPer; ++j) {
    const int i = min(part + kParts * j, kD - 1) * R + rc;
    v[0][j] = EF[i];
    v[1][j] = KF[i];
    b[j] = B[i];
  }
#pragma unroll
  for (int j = 0; j < 2; ++j) w[j] = Wrad[min(part + kParts * j, n_radial - 1) * R + rc];
  if (part == 0) sG[0][rank] = sG[1][rank] = sCol[0][rank] = sCol[1][rank] = sCol[2][rank] = kNone;
  if (tid < 3) sTop[tid] = kNone;
  if (tid < 18) sMax[tid] = 0;
  __syncthreads();
  // exponents of the ranks' columns of B and Wrad, and of KF
  auto raise = [&](int* p, int e) __attribute__((always_inline)) {
    if (in && e > kNone / 2) atomicMax(p + rank, e);
  };
  int eb = kNone, ek = kNone;
#pragma unroll
  for (int j = 0; j < kRowsPer; ++j) {
    const int k = part + kParts * j;
    if (k < kD) sF[0][k][rank] = v[0][j], sF[1][k][rank] = v[1][j];
    eb = max(eb, mag_exp(b[j])), ek = max(ek, mag_exp(v[1][j]));  // (a row past the last is the last)
  }
  raise(sG[0], eb);
  raise(sG[1], max(mag_exp(w[0]), mag_exp(w[1])));
  raise(sCol[1], ek);
  __syncthreads();
  // relative to the largest row; a row that adds nothing stays
  auto row_exp = [&](int q, int k) __attribute__((always_inline)) {
    const int e = sRow[q][k];
    return e == kNone ? 0 : e - sTop[q];
  };
  // EF's rows, each rank weighed by what else it multiplies, g and KF's column;
  // its columns then; and KF's by what EF has not taken
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    if (tid < kD * 32) {
      const int k = tid / 32;
      int m = kNone;
#pragma unroll
      for (int j = 0; j < kMost / 32; ++j) {
        const int r = (tid & 31) + 32 * j;
        const int e = mag_exp(sF[q][k][r]) + sG[0][r] + sG[1][r] + sCol[1 - q][r];
        if (r < R && e > kNone / 2) m = max(m, e);
      }
#pragma unroll
      for (int o = 16; o > 0; o >>= 1) m = max(m, __shfl_xor(m, o));
      if ((tid & 31) == 0) {
        sRow[q][k] = m;
        atomicMax(&sTop[q], m);
      }
    }
    __syncthreads();
    int e = kNone;
#pragma unroll
    for (int j = 0; j < kRowsPer; ++j) e = max(e, mag_exp(v[q][j]) - row_exp(q, min(part + kParts * j, kD - 1)));
    raise(sCol[2 * q], e);
    __syncthreads();
  }
  // a rank's column scales, if it adds something, and the largest with g's
  // exponents: |g| times a rank's factor 2^(share - most) is at most 25 * 16
  const int g_exp = sG[0][rank] + sG[1][rank];
  int share = sCol[0][rank] + sCol[2][rank], most = share + g_exp;
  if (most < kNone / 2) share = most = kNone;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) most = max(most, __shfl_xor(most, o));
  if (lane == 0 && wave < 2) atomicMax(&sTop[2], most);
  __syncthreads();
  most = sTop[2] == kNone ? 0 : sTop[2];
  auto scaled = [&](int q, int k, int r) __attribute__((always_inline)) {
    const int e = sCol[2 * q][r];
    return ldexpf(sF[q][k][r], 14 - row_exp(q, k) - (e == kNone ? 0 : e));
  };
  const MatOps O = mat_ops(RS);
  if (blockIdx.x == 0) {
    const int s = wave >> 1, l = lane & 31, r0 = 16 * s + 8 * (lane >> 5);
    if (s >= RS) return;
    float e[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) e[j] = l < kD && r0 + j < R ? scaled(wave & 1, l, r0 + j) : 0.f;
    if ((wave & 1) == 0) {
      float4* eo = reinterpret_cast<float4*>(out) + 2 * s * kWave + lane;
      eo[0] = make_float4(e[0], e[1], e[2], e[3]);
      eo[kWave] = make_float4(e[4], e[5], e[6], e[7]);
    } else {
      uint32_t u[2][4];
#pragma unroll
      for (int j = 0; j < 4; ++j) split_f16x2_pair(e[2 * j], e[2 * j + 1], u[0][j], u[1][j]);
      u32x4* ko = reinterpret_cast<u32x4*>(out + O.off_kf) + 2 * s * kWave + lane;
      ko[0] = u32x4{u[0][0], u[0][1], u[0][2], u[0][3]};
      ko[kWave] = u32x4{u[1][0], u[1][1], u[1][2], u[1][3]};
    }
    return;
  }
  // the largest of the scaled factors' row norms (sixteen threads a row) and of
  // g's bound per radial function; magnitudes compare as integers
  auto largest = [&](int* p, float m) __attribute__((always_inline)) { atomicMax(p, int(__float_as_uint(m))); };
  if (tid < 2 * kD * 16) {
    const int q = tid / (16 * kD), k = tid / 16 - q * kD;
    float n2 = 0.f;
#pragma unroll
    for (int j = 0; j < kMost / 16; ++j) {
      const int r = (tid & 15) + 16 * j;
      const float u = r < R ? scaled(q, k, r) : 0.f;
      n2 += fabsf(u) <= 16384.f ? u * u : 0.f;
    }
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) n2 += __shfl_xor(n2, o);
    if ((tid & 15) == 0) largest(&sMax[16 + q], n2);
  }
  {
    float n2 = 0.f;
    const int e = sG[0][rank] == kNone ? 0 : -sG[0][rank];
#pragma unroll
    for (int j = 0; j < kRowsPer; ++j) {
      const float u = part + kParts * j < kD ? ldexpf(b[j], e) : 0.f;
      n2 += fabsf(u) <= 1.f ? u * u : 0.f;
    }
    sPart[part][rank] = n2;
  }
  __syncthreads();
  {
    float n2 = 0.f;
#pragma unroll
    for (int p = 0; p < kParts; ++p) n2 += sPart[p][rank];
    const float n = 5.01f * sqrtf(n2);
    const int e = sG[1][rank] == kNone ? 0 : -sG[1][rank];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int q = part + kParts * j;
      const float u = ldexpf(fabsf(w[j]), e);
      float m = in && q < n_radial && share != kNone && u <= 1.f ? ldexpf(n * u, g_exp + share - most) : 0.f;
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
      if (lane == 0) largest(&sMax[q], m);
    }
  }
  __syncthreads();
  MatConst* c = reinterpret_cast<MatConst*>(out + O.off_const);
  if (tid < 16) c->bound[tid] = __uint_as_float(uint32_t(sMax[tid]));
  if (tid == 0) {
    c->e_fac = most - 28;
    int es = 0;
    (void)frexpf(sqrtf(__uint_as_float(uint32_t(sMax[16]))) * sqrtf(__uint_as_float(uint32_t(sMax[17]))) * 1.01f, &es);
    c->e_split = es < 14 ? 0 : es - 14;  // (at most 22: 128 ranks below 2^14 each)
  }
  if (tid < 16 * RS)
    reinterpret_cast<float*>(out + O.off_g)[tid] = share == kNone ? 0.f : ldexpf(1.f, min(share - most, 126));
  if (tid < 2 * kTile) {
    const int q = tid / kTile, k = tid % kTile;
    reinterpret_cast<int*>(out + (q ? O.off_rk : O.off_re))[k] = k < kD ? row_exp(q, k) : 0;
  }
}

template <bool BF, bool ATT, bool FG>
hipError_t dispatch(const EdgeArgs& a, hipStream_t s) {
  const bool r3 = a.R <= 96;
  if constexpr (BF) {
    if (a.C <= 128) return launch_mat<8, 4, true, false>(a, s);  // (mat_use: more than 96 ranks)
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

namespace mat_detail {
namespace {
int rank_steps(int R) { return 2 * ((R + kTile - 1) / kTile); }
}  // namespace
}  // namespace mat_detail

const int32_t* mat_row_exp(int R, const void* ops) {
  return reinterpret_cast<const int32_t*>(static_cast<const char*>(ops) +
                                          mat_detail::mat_ops(mat_detail::rank_steps(R)).off_rk);
}

hipError_t launch_mat_factor(int R, int n_radial, const float* EF, const float* KF, const float* B,
                             const float* radial_w, void* ops, hipStream_t s) {
  using namespace mat_detail;
  if (R < 1 || R > 128 || n_radial < 1 || n_radial > 16 || !EF || !KF || !B || !radial_w || !ops)
    return hipErrorInvalidValue;
  const int RS = rank_steps(R);
  if (size_t(mat_ops(RS).bytes) > edge_ef_bytes(kD, R)) return hipErrorInvalidValue;
  k_mat_factor<<<dim3(2), dim3(1024), 0, s>>>(R, RS, n_radial, EF, KF, B, radial_w,
                                                           static_cast<char*>(ops));
  return hipGetLastError();
}

hipError_t launch_cp_edge_mat(const EdgeArgs& a, hipStream_t s) {
  using namespace mat_detail;
  if (a.parts != 1 && a.parts != 2) return hipErrorInvalidValue;
  if (!mat_use(a.L, a.R, a.C, a.parts == 1, a.n_range) || a.n_range > a.E) return hipErrorInvalidValue;
  if (a.n_radial < 2 || a.n_radial > 16 || a.C > 256 || !a.ef_ops || (a.parts == 2 && !a.row_scale))
    return hipErrorInvalidValue;
  if (a.fa_global && (a.parts != 2 || a.alpha)) return hipErrorInvalidValue;
  if (a.alpha && (a.parts != 2 || a.n_heads < 1 || a.C % (kTile * a.n_heads) != 0)) return hipErrorInvalidValue;
  hipError_t e;
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
