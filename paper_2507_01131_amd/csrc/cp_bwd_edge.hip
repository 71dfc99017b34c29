// Backward with respect to the edge vectors, d > 32: what follows from
// dg_e (cp_bwd_dst_impl.hpp).  With g_e = v * rho, v = Y B, rho = Phi Wrad,
//   dv = dg * rho,  drho = dg * v,  dY = B dv,  dphi = Wrad drho,
//   grad r_e = J_Y(r_e)^T dY + (sum_q dphi_q phi'_q(|r_e|)) r_e/|r_e|.
// No sum runs over edges, so they are taken in the order of their ids, 32 at a
// time (two row tiles of 16x16x4 fp32 MFMA).  Bound by the latency of a
// chunk's phases.  A wave's operands of B and Wrad are the same for every
// chunk and stay in registers, which leaves room for one
// workgroup of eight waves a CU: 0.62 ms at 306 k edges, d = 49, R = 256; with
// 16 edges at a time 0.75; with two workgroups and the operands read from
// memory for every chunk 1.1 (spilled by the tighter register bound, 0.87).
#include "common.hpp"
#include "kernels.h"
#include "sh_device.hpp"

namespace tdn {
namespace bwd_detail {

constexpr int kRows = 16, kTiles = 2, kChunk = kRows * kTiles;  // edges of an MFMA tile, of a chunk

// LDS of the edge kernel, in floats: v and rho (the region then holds the rank
// tiles' shares of dY and dphi), Y (then dY), dY/dr, the radial basis, dphi.
struct EdgeSmem {
  int Rs, py, off_rho, off_y, off_j, off_phi, off_dphi, floats;
};
__host__ __device__ inline EdgeSmem edge_smem(int RT, int d, int n_radial) {
  EdgeSmem s{};
  s.Rs = RT * kTile + 4;  // the dY products read columns of v and rho
  s.py = (d + n_radial) | 1;
  s.off_rho = kChunk * s.Rs;
  const int v = 2 * kChunk * s.Rs, part = RT * kChunk * s.py;
  int o = v > part ? v : part;
  s.off_y = o;
  o += kChunk * d;
  s.off_j = o;
  o += kChunk * 3 * d;
  s.off_phi = o;
  o += kChunk * n_radial;
  s.off_dphi = o;
  o += kChunk * n_radial;
  s.floats = o;
  return s;
}

namespace {

constexpr int kEdgeWaves = 8, kEdgeWgs = 1;  // waves of a workgroup, workgroups of a CU
template <int L, int RT>
__global__ __launch_bounds__(kEdgeWaves* kWave) __attribute__((amdgpu_waves_per_eu(kEdgeWgs * 2))) void k_bwd_edge(
    BwdDstArgs a) {
  constexpr int d = (L + 1) * (L + 1), Rp = RT * kTile, Rs = Rp + 4;
  constexpr int kDg = kChunk * Rp / (kEdgeWaves * kWave);  // values of dg per thread
  extern __shared__ float smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g4 = lane >> 4, l16 = lane & 15;  // 16x16x4 MFMA operand coordinates
  const int nr = a.n_radial, R = a.R;
  const EdgeSmem S = edge_smem(RT, d, nr);
  const int py = S.py;
  float* sV = smem;
  float* sRho = smem + S.off_rho;
  float* sPart = smem;
  float* sY = smem + S.off_y;
  float* sDY = sY;
  float* sJ = smem + S.off_j;
  float* sPhi = smem + S.off_phi;
  float* sDPhi = smem + S.off_dphi;

  // the wave's operands of B and Wrad (its rank tile) stay in registers: rows
  // k, columns r for v and rho; rows r, columns k for dY and dphi
  constexpr int K = (d + 3) / 4, T = (d + 15) / 16;
  const int rt = wave;  // RT <= kEdgeWaves: one rank tile per wave at most
  float bv[K][2], bw[4][2], bt[8][T], wt[8];
  if (rt < RT) {
#pragma unroll
    for (int c2 = 0; c2 < 2; ++c2) {
      const int r = rt * kTile + 16 * c2 + l16, rc = min(r, R - 1);
#pragma unroll
      for (int s4 = 0; s4 < K; ++s4) {
        const int k = 4 * s4 + g4;
        const float v = a.Bf[min(k, d - 1) * R + rc];
        bv[s4][c2] = k < d && r < R ? v : 0.f;
      }
#pragma unroll
      for (int s4 = 0; s4 < 4; ++s4) {
        const int q = 4 * s4 + g4;
        const float v = a.radial_w[min(q, nr - 1) * R + rc];
        bw[s4][c2] = q < nr && r < R ? v : 0.f;
      }
    }
#pragma unroll
    for (int s4 = 0; s4 < 8; ++s4) {
      const int rr = rt * kTile + 4 * s4 + g4, rc = min(rr, R - 1);
#pragma unroll
      for (int t = 0; t < T; ++t) {
        const int k = 16 * t + l16;
        const float v = a.Bf[min(k, d - 1) * R + rc];
        bt[s4][t] = rr < R && k < d ? v : 0.f;
      }
      const float v = a.radial_w[min(l16, nr - 1) * R + rc];
      wt[s4] = rr < R && l16 < nr ? v : 0.f;
    }
  }

  for (int cb = blockIdx.x * kChunk; cb < a.E; cb += gridDim.x * kChunk) {
    const int n = min(kChunk, a.E - cb);
    float dg[kDg];
#pragma unroll
    for (int j = 0; j < kDg; ++j) {
      const int i = tid + j * kEdgeWaves * kWave, e = i / Rp, r = i - e * Rp;
      dg[j] = e < n && r < R ? a.dg[size_t(cb + e) * R + r] : 0.f;
    }
    __syncthreads();
    // harmonics and Jacobian per (edge, order m) column; radial basis per
    // (edge, function)
    for (int t = tid; t < n * (L + 1); t += blockDim.x) {
      const int e = t / (L + 1), m = t - e * (L + 1);
      const float* ev = a.edge_vec + 3 * size_t(cb + e);
      const float vx = ev[0], vy = ev[1], vz = ev[2];
      const float inv = 1.f / sqrtf(vx * vx + vy * vy + vz * vz);
      sh_unit_jacobian_column(a.L, m, vx * inv, vy * inv, vz * inv, inv, sY + e * d, sJ + e * 3 * d);
    }
    for (int t = int(blockDim.x) - 1 - tid; t < n * nr; t += blockDim.x) {
      const int e = t / nr, q = t - e * nr;
      const float* ev = a.edge_vec + 3 * size_t(cb + e);
      sPhi[t] = radial_phi(sqrtf(ev[0] * ev[0] + ev[1] * ev[1] + ev[2] * ev[2]), q, a.sigma);
    }
    __syncthreads();
    // v = Y B and rho = Phi Wrad on 16x16x4 fp32 MFMA (rows: 16 edges;
    // columns: two 16-rank halves of one 32-rank tile per wave at a
    // time; contraction over k < d, then over the radial functions)
    if (rt < RT) {
#pragma unroll
      for (int u = 0; u < kTiles; ++u) {
        const int er = u * kRows + l16;
        f32x4 tv[2] = {f32x4{}, f32x4{}}, tr[2] = {f32x4{}, f32x4{}};
#pragma unroll
        for (int s4 = 0; s4 < K; ++s4) {
          const int k = 4 * s4 + g4;
          const float av = (er < n && k < d) ? sY[er * d + k] : 0.f;
#pragma unroll
          for (int c2 = 0; c2 < 2; ++c2) tv[c2] = mfma16f32(av, bv[s4][c2], tv[c2]);
        }
#pragma unroll
        for (int s4 = 0; s4 < 4; ++s4) {
          const int q = 4 * s4 + g4;
          const float av = (er < n && q < nr) ? sPhi[er * nr + q] : 0.f;
#pragma unroll
          for (int c2 = 0; c2 < 2; ++c2)
            if (4 * s4 < nr) tr[c2] = mfma16f32(av, bw[s4][c2], tr[c2]);
        }
#pragma unroll
        for (int c2 = 0; c2 < 2; ++c2)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int e = u * kRows + 4 * g4 + i, r = rt * kTile + 16 * c2 + l16;
            if (e < n) {
              sV[e * Rs + r] = tv[c2][i];
              sRho[e * Rs + r] = tr[c2][i];
            }
          }
      }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kDg; ++q) {
      const int i = tid + q * kEdgeWaves * kWave, e = i / Rp, r = i - e * Rp, j = e * Rs + r;
      if (e < n) {
        const float dv = dg[q] * sRho[j], drho = dg[q] * sV[j];
        sV[j] = dv;
        sRho[j] = drho;
        if (a.drho && r < R) a.drho[size_t(cb + e) * R + r] = drho;  // for the radial-weight gradient
      }
    }
    __syncthreads();
    // dY = dV B^T (columns k < d: up to four 16-column tiles) and dphi =
    // dRho Wrad^T (columns q < n_radial <= 16: one tile) on 16x16x4 fp32
    // MFMA, contraction over one rank tile of 32 per wave (eight steps); the
    // per-tile partials go to the v/rho region and are summed over the rank
    // tiles in a fixed order.
    {
      f32x4 pt[kTiles][5];
      if (rt < RT) {
#pragma unroll
        for (int u = 0; u < kTiles; ++u) {
          const int er = u * kRows + l16;
#pragma unroll
          for (int t = 0; t < 5; ++t) pt[u][t] = f32x4{};
#pragma unroll
          for (int s4 = 0; s4 < 8; ++s4) {
            const int rr = rt * kTile + 4 * s4 + g4;
            const float a_v = er < n ? sV[er * Rs + rr] : 0.f;
            const float a_r = er < n ? sRho[er * Rs + rr] : 0.f;
#pragma unroll
            for (int t = 0; t < T; ++t) pt[u][t] = mfma16f32(a_v, bt[s4][t], pt[u][t]);
            pt[u][4] = mfma16f32(a_r, wt[s4], pt[u][4]);
          }
        }
      }
      __syncthreads();  // every wave has read dv and drho
      if (rt < RT) {
#pragma unroll
        for (int u = 0; u < kTiles; ++u)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            float* o = sPart + (rt * kChunk + u * kRows + 4 * g4 + i) * py;
#pragma unroll
            for (int t = 0; t < T; ++t)
              if (16 * t + l16 < d) o[16 * t + l16] = pt[u][t][i];
            if (l16 < nr) o[d + l16] = pt[u][4][i];
          }
      }
      __syncthreads();
      for (int i = tid; i < n * (d + nr); i += blockDim.x) {
        const int e = i / (d + nr), c = i - e * (d + nr);
        float sum = 0.f;
        for (int w = 0; w < RT; ++w) sum += sPart[(w * kChunk + e) * py + c];
        if (c < d)
          sDY[e * d + c] = sum;
        else
          sDPhi[e * nr + c - d] = sum;
      }
    }
    __syncthreads();
    // the gradient on sixteen threads an edge, their shares added in a fixed
    // order
    if (tid < kChunk * 16) {
      const int e = min(tid >> 4, n - 1);
      const float* ev = a.edge_vec + 3 * size_t(cb + e);
      const float vx = ev[0], vy = ev[1], vz = ev[2];
      const float rn = sqrtf(vx * vx + vy * vy + vz * vz);
      float g[3] = {0.f, 0.f, 0.f}, dr = 0.f;
      for (int k = l16; k < d; k += 16) {
        const float dy = sDY[e * d + k];
#pragma unroll
        for (int x = 0; x < 3; ++x) g[x] += dy * sJ[e * 3 * d + 3 * k + x];
      }
      if (l16 < nr) dr = sDPhi[e * nr + l16] * (-radial_t(rn, l16, a.sigma) / a.sigma) * sPhi[e * nr + l16];
#pragma unroll
      for (int o = 8; o > 0; o >>= 1) {
#pragma unroll
        for (int x = 0; x < 3; ++x) g[x] += __shfl_xor(g[x], o);
        dr += __shfl_xor(dr, o);
      }
      if ((tid >> 4) < n && l16 < 3) {
        const float v = l16 == 0 ? vx : (l16 == 1 ? vy : vz);
        a.grad_vec[3 * size_t(cb + e) + l16] = (l16 == 0 ? g[0] : (l16 == 1 ? g[1] : g[2])) + dr * v * (1.f / rn);
      }
    }
  }
}

template <int L, int RT>
hipError_t launch_edge_k(const BwdDstArgs& a, int lds, hipStream_t s) {
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_bwd_edge<L, RT>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (e != hipSuccess) return e;
  const int chunks = (a.E + kChunk - 1) / kChunk, most = kEdgeWgs * device_cus();
  k_bwd_edge<L, RT><<<dim3(chunks < most ? chunks : most), dim3(kEdgeWaves * kWave), lds, s>>>(a);
  return hipGetLastError();
}
}  // namespace

// The edge kernel after the dg kernel.
hipError_t launch_edge(const BwdDstArgs& a, hipStream_t s) {
  const size_t lds = size_t(edge_smem((a.R + kTile - 1) / kTile, a.d, a.n_radial).floats) * 4;
  if (lds > 160 * 1024 || a.R > kEdgeWaves * kTile || a.L < 5 || a.L > 6 || a.n_radial > 16) return hipErrorInvalidValue;
  switch ((a.L - 5) * 8 + (a.R + kTile - 1) / kTile) {
#define TDN_EDGE_CASE(RTV)                                 \
  case RTV: return launch_edge_k<5, RTV>(a, int(lds), s); \
  case 8 + RTV: return launch_edge_k<6, RTV>(a, int(lds), s);
    TDN_EDGE_CASE(1)
    TDN_EDGE_CASE(2)
    TDN_EDGE_CASE(3)
    TDN_EDGE_CASE(4)
    TDN_EDGE_CASE(5)
    TDN_EDGE_CASE(6)
    TDN_EDGE_CASE(7)
    TDN_EDGE_CASE(8)
#undef TDN_EDGE_CASE
    default: return hipErrorInvalidValue;
  }
}

}  // namespace bwd_detail
}  // namespace tdn
