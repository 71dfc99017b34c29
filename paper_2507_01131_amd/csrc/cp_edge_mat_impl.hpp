// The edge pass of degree L = 4 through per-edge matrices.
//
// Every edge's message before the channel mix is a matrix times the gathered
// row, z_e = K_e feat[gather[e]] with
//   K_e[k, i] = sum_r EF[k, r] g_e[r] KF[i, r]          ([25, 25]),
// and the sum over a segment adds the z_e themselves, so no output factor is
// applied to the segment's sum.  On 32x32x16 MFMA over two-part fp16 splits an
// edge takes 3 R/16 products for K_e and 6 per 32 channels for K_e x: 48 at
// R = C = 128, against 80 for the rank form of cp_edge_impl.hpp (5 per 32
// ranks and 32 channels) plus its epilogue.
//
// A workgroup has four teams of two waves, one team per SIMD, each with a
// range of the sorted edges: the builder forms the range's matrices, two edges
// at a time, and the applier multiplies them with the gathered rows and keeps
// the segment's [25, C] sum in fp32 registers.  The two kinds of work overlap
// because they are different waves of one SIMD.  The matrices go through LDS,
// double-buffered, one workgroup barrier per two edges.
//
// What bounds it, at 3200 nodes, 151 k edges, R = C = 128 (rank form 426 us,
// this one 307): a builder alone takes 230 us (a wave by itself issues a vector
// instruction every eight cycles, and forming and splitting EF g takes 250 an
// edge), an applier alone 200 us (the rows, 14 KB an edge from the L2, arrive
// one edge later).  Two builders per applier leave the applier's rows too few
// registers (408 us); one builder and two appliers of half the columns read
// the matrices twice (387 us); all edges' products added in the MFMA
// accumulators at a scale per segment took 319 us, with half again the error.
//
// Builder.  K_e^T = KF (EF g)^T on MFMA: A operand KF (rows i), constant, fp16
// parts in registers; B operand EF[k, r] g_e[r] for this lane's k and eight
// ranks per step, formed in fp32 from registers and split.  The accumulators
// (rows i, column k = lane) are split again and are, as they stand, the A
// operand of the applier's product: registers 8 q .. 8 q + 7 of lane half h
// are the K slots i = acc_krow(q, h, 0..7) of row k, and the rows are laid out
// in that order (launch_feature_layout_mat).  While it builds 16 edges, a
// builder also forms the next 16 edges' g = (Y B) * (Phi Wrad), a little at
// each step: harmonics and radial basis at the first, then a 16-rank tile on
// fp32 MFMA at a time.
//
// Scales, all exact powers of two.  An fp16 operand holds 28 binary orders at
// full precision, so what varies between rows, ranks and edges is taken out of
// it.  EF and KF are scaled per row, by what their ranks can add to K_e there,
// then per rank (column, to [2^13, 2^14)); a rank's g_e is multiplied by its
// column scales; and each edge's g is brought below 1 by a bound with a term per
// radial function q, sum_q phi_q max_r 5 |B_r| |Wrad[q, r]| scale_r (the
// harmonics' squares add up to 25), or by its largest value where the bound is
// far above it.  K_e is split (fp32 problems) at max_k |EF_k| max_i |KF_i| of the
// scaled rows.  KF's row scales come back in the feature rows
// (launch_feature_layout_mat), EF's where a segment's sum is stored, and the
// others in one exponent per edge: its product is added in fp32 with 2^that, its
// row's scale and, in the attention block, its head's weight.  bf16 problems:
// EF g and KF in one fp16 part, K_e rounded to bf16 with its edge's exponent, the
// sum in the MFMA accumulators.
#pragma once

#include <type_traits>
#include <utility>

#include "common.hpp"
#include "kernels.h"
#include "sh_device.hpp"

namespace tdn {
namespace mat_detail {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x3 __attribute__((ext_vector_type(3)));
typedef u32x3 u32x3_a4 __attribute__((aligned(4)));

__device__ __forceinline__ f32x16 mfma_bf16(u32x4 a, u32x4 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0,
                                                 0, 0);
}
__device__ __forceinline__ f32x16 mfma_f16(u32x4 a, u32x4 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0,
                                                0);
}

// f(0), ..., f(N - 1) with constant arguments.
template <int... I, typename F>
__device__ __forceinline__ void static_for_seq(std::integer_sequence<int, I...>, F&& f) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_seq(std::make_integer_sequence<int, N>{}, f);
}

constexpr int kL = 4, kD = 25;
constexpr int kTeams = 4;   // teams of a workgroup, one per SIMD
constexpr int kRoles = 2;   // a builder and an applier
constexpr int kGeo = 16;    // edges per geometry step
constexpr int kSub = 2;     // edges per barrier

// LDS of a workgroup, in floats: the matrices [team][2][kSub][2 parts] of
// [64 lanes] x 16 bytes, the exponents of their products, the output rows'
// exponents [32], g [team][2][16][Rp], and per team Y [16][29], Phi [16][17] and
// the exponent per edge of two geometry steps.
struct MatSmem {
  int off_s, off_re, off_g, off_team, y, phi, exp, team, floats;
};
__host__ __device__ constexpr MatSmem mat_smem(int RS, bool bf) {
  MatSmem s{};
  int o = kTeams * 2 * kSub * (bf ? 2 : 4) * kWave * 4;
  s.off_s = o;
  o += kTeams * 2 * kSub;
  s.off_re = o;
  o += kTile;
  s.off_g = o;
  o += kTeams * 2 * kGeo * RS * 16;
  s.off_team = o;
  s.y = 0;
  s.phi = s.y + kGeo * 29;
  s.exp = s.phi + kGeo * 17;
  s.team = s.exp + 2 * kGeo;
  s.floats = o + kTeams * s.team;
  return s;
}

__device__ constexpr float kRecip[5] = {1.f, 1.f / 2.f, 1.f / 3.f, 1.f / 4.f, 1.f / 5.f};
// Order m (and -m) of the harmonics of a unit vector, l = m .. 4.
__device__ __forceinline__ void sh_column(int m, float x, float y, float z, float* Y) {
  float re = 1.f, im = 0.f, p = 1.f, p_prev = 0.f;
  for (int k = 0; k < m; ++k) {
    const float re2 = re * x - im * y;
    im = re * y + im * x;
    re = re2;
    p *= float(2 * k + 1);
  }
  for (int l = m; l <= kL; ++l) {
    const float c = kShNorm.v[l][m] * p;
    Y[l * l + l + m] = c * re;
    if (m > 0) Y[l * l + l - m] = c * im;
    // t / (l - m + 1), rounded once: the reciprocal's product and its remainder
    const float t = float(2 * l + 1) * z * p - float(l + m) * p_prev, q = t * kRecip[l - m];
    const float pn = fmaf(fmaf(-q, float(l - m + 1), t), kRecip[l - m], q);
    p_prev = p;
    p = pn;
  }
}

// What the launch's factor kernel leaves in ef_ops, in bytes: EF's operands,
// KF's, then MatConst, the ranks' factors of g [16 RS] and the exponents of the
// output's and the features' rows [32] each, relative to the largest.
struct MatOps {
  int off_kf, off_const, off_g, off_re, off_rk, bytes;
};
__host__ __device__ constexpr MatOps mat_ops(int RS) {
  MatOps o{};
  o.off_kf = RS * 2048;
  o.off_const = 2 * o.off_kf;
  o.off_g = o.off_const + 80;
  o.off_re = o.off_g + RS * 64;
  o.off_rk = o.off_re + kTile * 4;
  o.bytes = o.off_rk + kTile * 4;
  return o;
}
// bound: of |g| times its rank's factor, per radial function; e_fac: a product
// of the scaled factors and g times 2^e_fac is the true one; e_split: |K_e| of the
// scaled factors (|g| < 1) is at most 2^(14 + e_split).
struct MatConst {
  float bound[16];
  int e_fac, e_split;
};

// RS: rank steps of 16.  NT: channel tiles of 32 per applier (the columns of
// blockIdx.y).  ATT: every edge's message weighted per head (fp32 problems).
// FG: the measurement ablation whose builder reads its factor operands from
// memory for every edge.
template <int RS, int NT, bool BF, bool ATT, bool FG = false>
__global__ __launch_bounds__(kRoles* kTeams* kWave)
__attribute__((amdgpu_waves_per_eu(kRoles))) void k_cp_edge_mat(EdgeArgs a) {
  constexpr int P = BF ? 1 : 2;
  constexpr int KQ = 2 * P;  // 16-byte words per lane of a matrix
  constexpr int Rp = RS * 16;
  constexpr int kSteps = kGeo / kSub;        // barriers per geometry step
  constexpr int kTileSteps = RS / 2;  // of which with rank tiles of the next one
  static_assert(kTileSteps < kSteps && RS % 2 == 0, "the next edges' tiles fit one step");
  extern __shared__ __align__(16) float smem[];
  const int nr = a.n_radial, R = a.R, C = a.C, E = a.E;
  constexpr MatSmem S = mat_smem(RS, BF);
  u32x4* sK = reinterpret_cast<u32x4*>(smem);
  int* sS = reinterpret_cast<int*>(smem + S.off_s);  // exponents of the products
  int* sRe = reinterpret_cast<int*>(smem + S.off_re);
  // (the wave's number in a scalar register: everything that follows from it,
  // its range, positions and branches, is uniform)
  const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int h = lane >> 5, l32 = lane & 31;
  const int team = wave & (kTeams - 1), role = wave / kTeams;  // 0: the builder
  float* sG = smem + S.off_g + team * 2 * kGeo * Rp;
  float* sT = smem + S.off_team + team * S.team;

  const int b = xcd_remap(blockIdx.x, gridDim.x);
  const int range = b * kTeams + team;
  auto bound = [&](int r) { return int(int64_t(min(r, a.n_range)) * E / a.n_range); };
  const int lo = bound(range), hi = bound(range + 1);
  // barriers of the workgroup: its longest range
  int most = 0;
#pragma unroll
  for (int q = 0; q < kTeams; ++q) most = max(most, bound(b * kTeams + q + 1) - bound(b * kTeams + q));
  const int n_sub = (most + kSub - 1) / kSub;
  constexpr MatOps O = mat_ops(RS);
  const char* __restrict__ ops = static_cast<const char*>(a.ef_ops);
  const u32x4* __restrict__ kfp = reinterpret_cast<const u32x4*>(ops + O.off_kf) + lane;
  if (threadIdx.x < kTile) sRe[threadIdx.x] = reinterpret_cast<const int*>(ops + O.off_re)[threadIdx.x];

  if (role == 0) {
    float* sY = sT + S.y;
    float* sPhi = sT + S.phi;
    int* sExp = reinterpret_cast<int*>(sT + S.exp);
    const MatConst* __restrict__ mc = reinterpret_cast<const MatConst*>(ops + O.off_const);
    const float* __restrict__ gm = reinterpret_cast<const float*>(ops + O.off_g);
    // EF, this lane's row k = l32 and ranks 16 s + 8 h + j; KF, row i = l32
    const float4* __restrict__ efp = static_cast<const float4*>(a.ef_ops) + lane;
    float ef[RS * 8];
    u32x4 kf[RS][P];
    auto load_step = [&](int s, int at) __attribute__((always_inline)) {
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const float4 v = efp[(2 * s + q) * kWave + at];
        ef[8 * s + 4 * q] = v.x, ef[8 * s + 4 * q + 1] = v.y, ef[8 * s + 4 * q + 2] = v.z, ef[8 * s + 4 * q + 3] = v.w;
      }
#pragma unroll
      for (int p = 0; p < P; ++p) kf[s][p] = kfp[(2 * s + p) * kWave + at];
    };
    if constexpr (!FG)
#pragma unroll
      for (int s = 0; s < RS; ++s) load_step(s, 0);
    const int ge = lane & 15, gq = lane >> 4;
    // the next 16 edges' vectors, a geometry step ahead
    float vx = 0.f, vy = 0.f, vz = 1.f;
    auto fetch = [&](int p) __attribute__((always_inline)) {
      const int eid = a.perm[min(p + ge, E - 1)];
      vx = a.edge_vec[3 * size_t(eid)];
      vy = a.edge_vec[3 * size_t(eid) + 1];
      vz = a.edge_vec[3 * size_t(eid) + 2];
    };
    float mq[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) mq[q] = mc->bound[gq + 4 * q];
    const int e_fac = mc->e_fac, e_split = mc->e_split;
    float top[4];  // the largest |g| that this lane formed for edges 4 gq + i
    // harmonics, radial basis and scales of the 16 edges from p on, geometry
    // step number gi
    auto geometry = [&](int p, int gi) __attribute__((always_inline)) {
      const float len = sqrtf(vx * vx + vy * vy + vz * vz);
      {
        const float inv = 1.f / len;
        const float ux = vx * inv, uy = vy * inv, uz = vz * inv;
        for (int m = gq; m <= kL; m += 4) sh_column(m, ux, uy, uz, sY + ge * 29);
        if (gq == 1) sY[ge * 29 + 25] = sY[ge * 29 + 26] = sY[ge * 29 + 27] = 0.f;
      }
      {
        float ph[4], sum = 0.f;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          ph[q] = gq + 4 * q < nr ? radial_phi(len, gq + 4 * q, a.sigma) : 0.f;
          sum += ph[q] * mq[q];
        }
        sum += __shfl_xor(sum, 16);
        sum += __shfl_xor(sum, 32);
        int e = 0;
        (void)frexpf(sum, &e);
        e = sum > 0.f && sum < 3.0e38f ? max(e, -120) : 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) sPhi[ge * 17 + gq + 4 * q] = ldexpf(ph[q], -e);
        if (gq == 0) sExp[(gi & 1) * kGeo + ge] = e + e_fac + (BF ? 0 : e_split);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) top[i] = 0.f;
      if (p + kGeo < hi) fetch(p + kGeo);
    };
    // g, times its ranks' factors, of 16 edges and the 16 ranks of each tile from
    // t0 on (rows: edges, columns: ranks)
    auto rank_tiles = [&](int t0, int n, int gi) __attribute__((always_inline)) {
      const char* __restrict__ bp = reinterpret_cast<const char*>(a.Bf);
      const char* __restrict__ wp = reinterpret_cast<const char*>(a.radial_w);
      uint32_t bk[7], wk[4];  // byte offsets of the lane's rows
#pragma unroll
      for (int s = 0; s < 7; ++s) bk[s] = uint32_t(min(4 * s + gq, kD - 1) * R) * 4;  // (Y is zero from kD on)
#pragma unroll
      for (int s = 0; s < 4; ++s) wk[s] = uint32_t(min(4 * s + gq, nr - 1) * R) * 4;  // (Phi from n_radial on)
#pragma unroll 2
      for (int t = t0; t < t0 + n; ++t) {
        const uint32_t r = t * 16 + ge, rc = uint32_t(min(int(r), R - 1)) * 4;
        float bo[7], wo[4];
#pragma unroll
        for (int s = 0; s < 7; ++s) bo[s] = *reinterpret_cast<const float*>(bp + (bk[s] + rc));
#pragma unroll
        for (int s = 0; s < 4; ++s) wo[s] = *reinterpret_cast<const float*>(wp + (wk[s] + rc));
        const float m = gm[r];  // (zero from R on)
        f32x4 Ty = f32x4{}, Tr = f32x4{};
#pragma unroll
        for (int s = 0; s < 7; ++s) {
          Ty = mfma16f32(sY[ge * 29 + 4 * s + gq], bo[s], Ty);
          if (s < 2) Tr = mfma16f32(sPhi[ge * 17 + 4 * s + gq], wo[s], Tr);
        }
        if (nr > 8) {
          Tr = mfma16f32(sPhi[ge * 17 + 8 + gq], wo[2], Tr);
          Tr = mfma16f32(sPhi[ge * 17 + 12 + gq], wo[3], Tr);
        }
        float* o = sG + ((gi & 1) * kGeo + 4 * gq) * Rp + r;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float v = Ty[i] * (Tr[i] * m);
          top[i] = fmaxf(top[i], fabsf(v));
          o[i * Rp] = v;
        }
      }
    };
    // An edge whose g stays below 2^-6 (2^-14 in bf16 problems; harmonics that
    // vanish, weights that cancel) has it brought to [1/2, 1) by its largest; a
    // zero or non-finite one stays.  One edge at a time: there are few.
    auto level = [&](int gi) __attribute__((always_inline)) {
      unsigned long long low = 0;  // bit 16 gq + i: edge 4 gq + i
#pragma unroll
      for (int i = 0; i < 4; ++i) {  // (an edge's 16 lanes are 16 bits of the ballot)
        const unsigned long long b = __ballot(top[i] >= (BF ? 0x1p-14f : 0x1p-6f));
        low |= ((b - 0x0001000100010001ull) & ~b & 0x8000800080008000ull) >> (15 - i);
      }
      while (low) {
        const int at = __builtin_ctzll(low), e = (gi & 1) * kGeo + (at >> 4) * 4 + (at & 15);
        low &= low - 1;
        float* gp = sG + e * Rp + 2 * min(lane, Rp / 2 - 1);
        const float v0 = gp[0], v1 = gp[1];
        float mx = fmaxf(fabsf(v0), fabsf(v1));
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
        int x = 0;
        if (mx > 0.f && mx <= 3.4028234e38f) (void)frexpf(mx, &x);
        if (lane < Rp / 2) gp[0] = ldexpf(v0, -x), gp[1] = ldexpf(v1, -x);
        if (lane == 0) sExp[e] += x;
      }
    };
    const float split = ldexpf(1.f, -e_split);
    auto build = [&](int i, int gi, int buf, int slot) __attribute__((always_inline)) {
      const float4* gp = reinterpret_cast<const float4*>(sG + ((gi & 1) * kGeo + i) * Rp + 8 * h);
      f32x16 K = f32x16{};
      int at = 0;
      if constexpr (FG) asm volatile("" : "+v"(at));  // (the loads stay in the loop over edges)
#pragma unroll
      for (int s = 0; s < RS; ++s) {
        if constexpr (FG) load_step(s, at);
        const float4 g0 = gp[4 * s], g1 = gp[4 * s + 1];
        const float gv[8] = {g0.x, g0.y, g0.z, g0.w, g1.x, g1.y, g1.z, g1.w};
        uint32_t w[2][4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float t0 = ef[8 * s + 2 * q] * gv[2 * q], t1 = ef[8 * s + 2 * q + 1] * gv[2 * q + 1];
          if constexpr (BF)
            w[0][q] = pack_f16x2_rne(t0, t1);
          else
            split_f16x2_pair(t0, t1, w[0][q], w[1][q]);
        }
        const u32x4 hi4 = {w[0][0], w[0][1], w[0][2], w[0][3]};
        if constexpr (!BF) {
          const u32x4 lo4 = {w[1][0], w[1][1], w[1][2], w[1][3]};
          K = mfma_f16(kf[s][1], hi4, K);
          K = mfma_f16(kf[s][0], lo4, K);
        }
        K = mfma_f16(kf[s][0], hi4, K);
      }
      const int ex = sExp[(gi & 1) * kGeo + i];
      auto scaled = [&](float v) { return BF ? ldexpf(v, ex) : v * split; };
      u32x4* o = sK + ((team * 2 + buf) * kSub + slot) * (KQ * kWave) + lane;
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        uint32_t w[2][4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float x0 = scaled(K[8 * q + 2 * j]), x1 = scaled(K[8 * q + 2 * j + 1]);
          if constexpr (BF)
            w[0][j] = pack_bf16x2_rne(x0, x1);
          else
            split_f16x2_pair(x0, x1, w[0][j], w[1][j]);
        }
#pragma unroll
        for (int p = 0; p < P; ++p) o[(p * 2 + q) * kWave] = u32x4{w[p][0], w[p][1], w[p][2], w[p][3]};
      }
      if constexpr (!BF)
        if (lane == 0) sS[(team * 2 + buf) * kSub + slot] = ex;
    };
    fetch(lo);
    if (lo < hi) geometry(lo, 0);
    lds_barrier();
    if (lo < hi) {
      rank_tiles(0, RS, 0);
      level(0);
    }
    lds_barrier();
    for (int j = 0; j < n_sub; ++j) {
      const int p = lo + j * kSub, gi = j / kSteps, js = j % kSteps;
      const int pn = lo + (gi + 1) * kGeo;  // the next geometry step's first edge
      if (js == 0 && pn < hi) geometry(pn, gi + 1);
#pragma unroll 1
      for (int q = 0; q < kSub; ++q)
        if (p + q < hi) build(js * kSub + q, gi, j & 1, q);
      if (js >= 1 && js <= kTileSteps && pn < hi) rank_tiles(2 * (js - 1), 2, gi + 1);
      if (js == kTileSteps && pn < hi) level(gi + 1);
      lds_barrier();
    }
    lds_barrier();
    return;
  }

  // ---- applier
  constexpr int XB = 256 * 7 * P;  // bytes of a row's channel tile
  const int n_ct = (C + kTile - 1) / kTile;
  const int ct0 = int(blockIdx.y) * NT;
  const char* __restrict__ xs = static_cast<const char*>(a.feat);
  const size_t row_bytes = size_t(n_ct) * XB;
  struct XOps {
    u32x4 q0[NT][P];
    u32x3 q1[NT][P];  // (the fourth word of the operand is zero)
  };
  XOps x;
  auto quad = [](u32x3 v) __attribute__((always_inline)) { return u32x4{v[0], v[1], v[2], 0u}; };
  // a tile past the last reads the last one; its sums are not stored
  auto load_x = [&](int row, auto t) __attribute__((always_inline)) {
    const char* xt = xs + size_t(row) * row_bytes + min(ct0 + t, n_ct - 1) * XB;
    static_for<P>([&](auto p) {
      x.q0[t][p] = *reinterpret_cast<const u32x4*>(xt + uint32_t(p * 1024 + lane * 16));
      x.q1[t][p] = *reinterpret_cast<const u32x3_a4*>(xt + uint32_t(P * 1024 + p * 768 + lane * 12));
    });
  };
  f32x16 acc[NT];
  static_for<NT>([&](auto t) { acc[t] = f32x16{}; });
  int head[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) head[t] = ATT ? min(ct0 + t, n_ct - 1) * kTile / (C / a.n_heads) : 0;
  const size_t dC = size_t(kD) * C;
  auto flush = [&](float* dst) __attribute__((always_inline)) {
    static_for<NT>([&](auto t) {
      const int c = (ct0 + t) * kTile + l32;
      if (c < C) {
        float* dl = dst + (4 * h) * C + c;
#pragma unroll
        for (int v = 0; v < 16; ++v)
          if (acc_row(v, h) < kD) dl[(8 * (v >> 2) + (v & 3)) * C] = ldexpf(acc[t][v], sRe[acc_row(v, h)]);
      }
      acc[t] = f32x16{};
    });
  };

  // rows, segments and row scales of 64 edges, one per lane, the next 64
  // loaded ahead; bit i of `starts`: edge i opens a segment
  int rows = 0, segs = 0, rows_n = 0, segs_n = 0;
  float scs = 1.f, scs_n = 1.f, als[NT], als_n[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) als[t] = als_n[t] = 1.f;
  auto fetch = [&](int p) __attribute__((always_inline)) {
    const int pl = min(p + lane, E - 1), eid = a.perm[pl];
    rows_n = a.gather[eid];
    segs_n = a.key[eid];
    if constexpr (!BF) scs_n = a.row_scale[rows_n];
    if constexpr (ATT)
#pragma unroll
      for (int t = 0; t < NT; ++t) als_n[t] = a.alpha[size_t(pl) * a.n_heads + head[t]];
  };
  unsigned long long starts = 0;
  int last_seg = -1;
  auto advance = [&](int p) {
    rows = rows_n, segs = segs_n, scs = scs_n;
#pragma unroll
    for (int t = 0; t < NT; ++t) als[t] = als_n[t];
    int prev = __shfl_up(segs, 1);
    if (lane == 0) prev = last_seg;
    starts = __ballot(segs != prev);
    last_seg = __builtin_amdgcn_readlane(segs, 63);
    fetch(p + kWave);
  };
  auto row_at = [&](int i) {
    return i < kWave ? __builtin_amdgcn_readlane(rows, i) : __builtin_amdgcn_readlane(rows_n, i - kWave);
  };
  fetch(lo);
  // whether the first segment began before this range, the last goes on
  const bool open_lo = hi > lo && lo > 0 && a.key[a.perm[lo - 1]] == a.key[a.perm[lo]];
  const bool open_hi = hi > lo && hi < E && a.key[a.perm[hi]] == a.key[a.perm[hi - 1]];
  int cur = -1;
  bool first = true;
  float* part = a.partial + size_t(range) * 2 * dC;
  // The edge at position i of the current 64: its matrix k times its row,
  // every channel tile's row words replaced by those of the next edge once they
  // are used.
  auto apply = [&](int i, const u32x4* k, int ex) __attribute__((always_inline)) {
    if ((starts >> i) & 1) {
      if (cur >= 0) {
        flush(first && open_lo ? part : a.out + size_t(cur) * dC);
        first = false;
      }
      cur = __builtin_amdgcn_readlane(segs, i);
    }
    const int next = row_at(i + 1);
    if constexpr (BF) {
      static_for<NT>([&](auto t) {
        acc[t] = mfma_bf16(k[0], x.q0[t][0], acc[t]);
        acc[t] = mfma_bf16(k[1], quad(x.q1[t][0]), acc[t]);
        __builtin_amdgcn_sched_barrier(0);
        load_x(next, t);
        __builtin_amdgcn_sched_barrier(0);
      });
    } else {
      const float st = ldexpf(__uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(scs), i)), ex);
      f32x16 U[2];
      static_for<NT + 1>([&](auto tc) {
        constexpr int t = decltype(tc)::value;
        if constexpr (t < NT) {
          f32x16 u = mfma_f16(k[KQ / 2], x.q0[t][0], f32x16{});
          u = mfma_f16(k[KQ - 1], quad(x.q1[t][0]), u);
          u = mfma_f16(k[0], x.q0[t][P - 1], u);
          u = mfma_f16(k[1], quad(x.q1[t][P - 1]), u);
          u = mfma_f16(k[0], x.q0[t][0], u);
          U[t & 1] = mfma_f16(k[1], quad(x.q1[t][0]), u);
        }
        if constexpr (t > 0) {
          const float w =
              ATT ? st * __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(als[t - 1]), i)) : st;
#pragma unroll
          for (int v = 0; v < 16; ++v) acc[t - 1][v] += w * U[(t - 1) & 1][v];
        }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (t < NT) load_x(next, std::integral_constant<int, t>{});
        __builtin_amdgcn_sched_barrier(0);
      });
    }
  };
  lds_barrier();
  lds_barrier();
  lds_barrier();
  // a position's matrices and the exponent of its e-th edge
  auto step = [&](int j, auto e) __attribute__((always_inline)) {
    const u32x4* kp = sK + ((team * 2 + (j & 1)) * kSub + e) * (KQ * kWave) + lane;
    u32x4 k[KQ];
#pragma unroll
    for (int q = 0; q < KQ; ++q) k[q] = kp[q * kWave];
    const int ex = BF ? 0 : __builtin_amdgcn_readfirstlane(sS[(team * 2 + (j & 1)) * kSub + e]);
    apply(((j * kSub) & (kWave - 1)) + e, k, ex);
  };
  const int n = max(hi - lo, 0);
  if (n > 0) {
    advance(lo);
    static_for<NT>([&](auto t) { load_x(row_at(0), t); });
  }
  int j = 0;
#pragma clang loop unroll(disable)
  for (; j < n / kSub; ++j) {
    if (j > 0 && ((j * kSub) & (kWave - 1)) == 0) advance(lo + j * kSub);
    static_for<kSub>([&](auto e) { step(j, e); });
    lds_barrier();
  }
  if (n % kSub != 0) {
    if (j > 0 && ((j * kSub) & (kWave - 1)) == 0) advance(lo + j * kSub);
    step(j, std::integral_constant<int, 0>{});
    lds_barrier();
    ++j;
  }
  for (; j < n_sub; ++j) lds_barrier();
  if (cur >= 0) flush(first && open_lo ? part : (open_hi ? part + dC : a.out + size_t(cur) * dC));
}

template <int RS, int NT, bool BF, bool ATT, bool FG = false>
hipError_t launch_mat(const EdgeArgs& a, hipStream_t s) {
  const size_t lds = size_t(mat_smem(RS, BF).floats) * 4;
  auto k = k_cp_edge_mat<RS, NT, BF, ATT, FG>;
  const hipError_t e =
      hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
  if (e != hipSuccess) return e;
  const int n_ct = (a.C + kTile - 1) / kTile;
  k<<<dim3((a.n_range + kTeams - 1) / kTeams, (n_ct + NT - 1) / NT), dim3(kRoles * kTeams * kWave), lds, s>>>(a);
  return hipGetLastError();
}

}  // namespace mat_detail
}  // namespace tdn
