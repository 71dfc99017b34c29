// Backward of the CP tensor-product layer with respect to the edge vectors,
// d > 32: the cotangent of g_e (d <= 32 takes the factored forms in
// cp_bwd_dst2_impl.hpp and cp_bwd_sg_impl.hpp; what follows from dg is
// cp_bwd_edge.hip).
//
// With Gz = grad_out W^T and Gh_t = D^T Gz[t] (per destination node, [R, C]),
// the cotangent of g_e (eq. approximate, Sec. 3.1) is
//   dg_e[r] = sum_c Gh_t[r, c] (A^T x[s_e])[r, c] = sum_k A[k, r] P_e[k, r],
//   P_e = x[s_e] Gh_t^T   ([d, R], contraction over the C channels).
//
// A workgroup takes several segments, one after the other; each wave takes one
// 32-row k tile and a pair of 32-rank tiles, whose Gh^T tiles are formed once a
// segment (fp32 MFMA, K = d; one tile each by the two waves of a pair, exchanged
// through LDS); in accumulator layout lane l holds
// Gh^T[ct*32 + acc_row(v, l/32)][rt*32 + l%32], so registers 8q .. 8q+7 are the B
// operand of one 32x32x16 step of P_e = x[s_e] Gh^T that contracts channels
// ct*32 + 16q + 8(i/4) + 4h + i%4 (i = 0..7) in half-wave h.  The x operand comes
// in that channel order from the xd layout (launch_direct_layout): per edge and
// channel tile one 16-byte load per k tile, K-step and part, one or two channel
// tiles ahead.
//
// Arithmetic.  fp32 problems: x[n] 2^-e_n and the wave's Gh^T tiles scaled by
// a power of two (largest magnitude to [2^13, 2^14)) are split into two fp16
// parts each (to 2^-22) and P_e sums the three part products with i + j <= 3
// on v_mfma_f32_32x32x16_f16, fp32 accumulation; dg carries both scales back
// (exactly).  bf16 problems: x is bf16 and Gh^T is rounded to bf16, one
// product on v_mfma_f32_32x32x16_bf16.  dg over the wave's k tile is a
// 32-term dot product with A (from LDS, in accumulator order) plus one
// cross-half add; the two k tiles' parts are added in a fixed order.
//
// What bounds it, at 4960 nodes, 306 k edges, d = 49, C = 128, R = 256: 384
// products an edge, 3.2 ms at the 1.2 PFLOP/s that a large fp16 product
// reaches; it takes 4.1 ms, 0.3 of them for Gh^T (0.6 while every wave formed
// both its tiles).  The edges' small products, which were in this kernel
// behind barriers of the one workgroup that its registers and LDS leave room
// for, took 2.0 ms there and take 0.6 in cp_bwd_edge.hip.
#pragma once

#include "common.hpp"
#include "kernels.h"

namespace tdn {

namespace bwd_detail {

constexpr int kChunk = 16;  // edges per buffer of dg

// LDS of the dg kernel, in floats: A in accumulator order, then two buffers of
// a chunk's dg over each k tile (the region also holds Gz[seg] while Gh^T is
// formed, then its tiles while waves exchange them).
struct DgSmem {
  int Rs, off_dg, floats;
};
__host__ __device__ inline DgSmem dg_smem(int RT, int MT, int d, int C, int shared_floats) {
  DgSmem s{};
  s.Rs = RT * kTile + 4;
  s.off_dg = MT * RT * 4 * kWave * 4;
  int n = 2 * MT * kChunk * s.Rs;
  if (n < d * C) n = d * C;
  if (n < shared_floats) n = shared_floats;
  s.floats = s.off_dg + n;
  return s;
}

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

template <bool BF>
__device__ __forceinline__ f32x16 mfma16(u32x4 a, u32x4 b, f32x16 c) {
  if constexpr (BF)
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c,
                                                   0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0,
                                                  0, 0);
}

// Waves of the workgroup: MT k tiles x ceil(RT / 2) pairs of rank tiles.
__host__ __device__ constexpr int direct_waves(int MT, int RT) { return MT * ((RT + 1) / 2); }

// Whether the two waves of a rank-tile pair form one Gh^T tile each (up to
// four channel tiles; beyond, the exchange would not fit the LDS), and the
// floats of the exchange: half a tile and an exponent per wave.
__host__ __device__ constexpr bool gh_shared(int MT, int NCT) { return MT == 2 && NCT <= 4; }
__host__ __device__ constexpr int gh_floats(int MT, int RT, int NCT, int P) {
  return gh_shared(MT, NCT) ? direct_waves(MT, RT) * (NCT * P * kWave * 4 + 1) : 0;
}

// dg of every edge, by edge id.
template <int MT, int RT, int NCT, bool BF>
__global__ __launch_bounds__(direct_waves(MT, RT)* kWave)
__attribute__((amdgpu_waves_per_eu(NCT == 8 ? 1 : 2))) void k_bwd_dg_direct(BwdDstArgs a) {
  constexpr int P = BF ? 1 : 2;  // 16-bit parts per operand value
  constexpr int NS = 2 * NCT;    // K-steps of 16 channels (xd blocks per part)
  constexpr int kSlots = NCT == 8 ? 2 : 4, kAhead = NCT == 8 ? 1 : 2;  // x steps held, loaded ahead
  extern __shared__ float smem[];
  const DgSmem S = dg_smem(RT, MT, a.d, a.C, gh_floats(MT, RT, NCT, P));
  constexpr int Rp = RT * kTile, Rs = Rp + 4;
  f32x4* sAl = reinterpret_cast<f32x4*>(smem);
  float* sDG = smem + S.off_dg;  // [2][MT][kChunk][Rs]: dg over each k tile

  // The workgroup's segments.  One for each, or almost two: every gridDim.x-th,
  // as a workgroup that takes one more than it has to takes the whole launch with
  // it (by edges, 50 segments: 205 us against 109; d = 36, C = R = 256, 500 on 256
  // workgroups: the force call 2220 us against 1920).  Else those that begin in
  // its share of the edges, which evens out their lengths (310 on 256: 1336 us
  // against 1379 that way).
  const int grid = gridDim.x;
  const bool few = a.n_seg <= grid || (4 * a.n_seg > 7 * grid && a.n_seg <= 2 * grid);
  auto first_at = [&](int p) {  // the first segment with offsets[seg] >= p
    int lo = 0, hi = a.n_seg;
    while (lo < hi) {
      const int mid = (lo + hi) / 2;
      if (a.offsets[mid] < p)
        lo = mid + 1;
      else
        hi = mid;
    }
    return lo;
  };
  const int b = xcd_remap(blockIdx.x, grid);
  const int item_lo = few ? int(blockIdx.x) : first_at(int(int64_t(b) * a.E / grid));
  const int item_hi = few ? a.n_seg : first_at(int(int64_t(b + 1) * a.E / grid));
  const int step = few ? grid : 1;
  if (item_lo >= item_hi) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = lane >> 5, l32 = lane & 31;
  const int d = a.d, C = a.C, R = a.R;
  // the P_e tiles of this wave: k tile kt, rank tiles 2j and 2j + 1; the first
  // is the one whose Gh^T tile this wave forms for both k tiles (kShare)
  constexpr bool kShare = gh_shared(MT, NCT);
  const int kt = wave % MT, pj = wave / MT, own = kShare ? kt : 0;
  int rtw[2];
  bool keep[2];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const int rt = 2 * pj + (t ^ own);
    keep[t] = rt < RT;  // a lone last tile runs twice; the copy is dropped
    rtw[t] = keep[t] ? rt : RT - 1;
  }

  // sAl[((kt*RT + rt)*4 + qq)*64 + lane'] = A[kt*32 + acc_row(4 qq + i, h')][rt*32 + l32']:
  // the A values lane' weighs its P accumulators with, one 16-byte read per quarter
  for (int t = tid; t < MT * RT * 4 * kWave; t += blockDim.x) {
    const int ln = t % kWave, q4 = t / kWave;
    const int qq = q4 % 4, krt = q4 / 4, rt = krt % RT, kt2 = krt / RT;
    const int r = rt * kTile + (ln & 31);
    f32x4 v;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int k = kt2 * kTile + acc_row(4 * qq + i, ln >> 5);
      v[i] = (k < d && r < R) ? a.A[k * R + r] : 0.f;
    }
    sAl[t] = v;
  }

  for (int item = item_lo; item < item_hi; item += step) {
    const int seg = few ? xcd_remap(item, a.n_seg) : item;
    const int e_begin = a.offsets[seg], e_end = a.offsets[seg + 1];
    if (e_begin == e_end) continue;
    // Gz[seg] staged in LDS ([d][C], coalesced float4 loads) in the dg region,
    // between the barriers that end its use
    __syncthreads();
    float* sGzf = sDG;
    {
      const f32x4* g4 = reinterpret_cast<const f32x4*>(a.Gz + size_t(seg) * d * C);
      for (int i = tid; i < d * C / 4; i += blockDim.x) reinterpret_cast<f32x4*>(sGzf)[i] = g4[i];
    }
    __syncthreads();
    // Gh^T tiles of the wave's two rank tiles, each scaled by its own power of
    // two (fp32 problems) and split: ghp[t][ct][q][p].  One D value per lane
    // and step feeds all channel tiles.
    u32x4 ghp[2][NCT][2][P];
    float gh_unscale[2] = {1.f, 1.f};
#pragma unroll
    for (int t = 0; t < (kShare ? 1 : 2); ++t) {
      const int r = rtw[t] * kTile + l32;
      f32x16 gh[NCT];
#pragma unroll
      for (int ct = 0; ct < NCT; ++ct) gh[ct] = f32x16{};
#pragma unroll 5
      for (int s2 = 0; s2 < (d + 1) / 2; ++s2) {
        const int k = 2 * s2 + h;
        const float bv = (k < d && r < R) ? a.D[k * R + r] : 0.f;
#pragma unroll
        for (int ct = 0; ct < NCT; ++ct) {
          const int cc = ct * kTile + l32;
          const float av = (k < d && cc < C) ? sGzf[k * C + cc] : 0.f;
          gh[ct] = mfma32(av, bv, gh[ct]);
        }
      }
      float sc = 1.f;
      if constexpr (!BF) {
        float mx = 0.f;
#pragma unroll
        for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
          for (int v = 0; v < 16; ++v) mx = fmaxf(mx, fabsf(gh[ct][v]));
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
        const int e = f16_split_exponent(mx);
        sc = ldexpf(1.f, -e);
        gh_unscale[t] = ldexpf(1.f, e);
      }
#pragma unroll
      for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          uint32_t w[P][4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float v0 = gh[ct][8 * q + 2 * i] * sc, v1 = gh[ct][8 * q + 2 * i + 1] * sc;
            if constexpr (BF)
              w[0][i] = pack_bf16x2_rne(v0, v1);
            else
              split_f16x2_pair(v0, v1, w[0][i], w[1][i]);
          }
#pragma unroll
          for (int p = 0; p < P; ++p) ghp[t][ct][q][p] = u32x4{w[p][0], w[p][1], w[p][2], w[p][3]};
        }
    }
    if constexpr (kShare) {
      // the other tile from the wave of the other k tile, half the channel tiles
      // at a time
      u32x4* sX = reinterpret_cast<u32x4*>(sDG);
      float* sE = sDG + direct_waves(MT, RT) * NCT * P * kWave * 4;
      constexpr int kHalf = NCT * P;  // words per lane and round: NCT / 2 tiles x 2 steps x P
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) {
        lds_barrier();  // Gz, or the first half, has been read
        if (hf == 0 && lane == 0) sE[wave] = gh_unscale[0];
#pragma unroll
        for (int i = 0; i < kHalf; ++i)
          sX[(wave * kHalf + i) * kWave + lane] = ghp[0][hf * (NCT / 2) + i / (2 * P)][i / P % 2][i % P];
        lds_barrier();
#pragma unroll
        for (int i = 0; i < kHalf; ++i)
          ghp[1][hf * (NCT / 2) + i / (2 * P)][i / P % 2][i % P] = sX[((wave ^ 1) * kHalf + i) * kWave + lane];
        if (hf == 0) gh_unscale[1] = sE[wave ^ 1];
      }
    }

    // x operand of channel tile ct for an edge row: xb[q][p] is lane (h, row
    // kt*32 + l32) of block (part p, K-step 2ct + q) of xd.  Rows past d are
    // clamped (their P rows meet A = 0).
    const char* __restrict__ xd = static_cast<const char*>(a.xc);
    const size_t node_bytes = size_t(P) * NS * 2 * d * 16;
    const int kr = kt * kTile + l32 < d ? kt * kTile + l32 : d - 1;
    const uint32_t lane_off = uint32_t((h * d + kr) * 16);
    auto load_step = [&](int row, int ct, u32x4 (&xb)[2][P]) {
      const char* base = xd + size_t(row) * node_bytes;
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int p = 0; p < P; ++p)
          xb[q][p] = *reinterpret_cast<const u32x4*>(base + lane_off + uint32_t((p * NS + 2 * ct + q) * 2 * d * 16));
    };

    __syncthreads();

    // P_e tiles and dg over this wave's k tile, edges in pairs so that the slot
    // of every (edge, ct) step is a compile-time choice; an odd last edge is
    // paired with a copy of itself whose result is dropped.  Rows and scales of
    // 64 edges, one per lane.
    for (int cb = e_begin; cb < e_end; cb += kWave) {
      const int n = min(kWave, e_end - cb);
      const int row_l = a.src[a.perm[cb + min(lane, n - 1)]];
      const float sc_l = BF ? 1.f : a.x_scale[row_l];
      auto row_at = [&](int e) { return __builtin_amdgcn_readlane(row_l, min(e, n - 1)); };
      u32x4 xb[kSlots][2][P];
      f32x16 pacc[2];
#pragma unroll
      for (int s = 0; s < kAhead; ++s) load_step(row_at(s / NCT), s % NCT, xb[s]);
      for (int e0 = 0; e0 < n; e0 += 2) {
        float* dgb = sDG + (((e0 / kChunk) & 1) * MT + kt) * kChunk * Rs;
#pragma unroll
        for (int s = 0; s < 2 * NCT; ++s) {
          const int e = e0 + s / NCT, ct = s % NCT;
          load_step(row_at(e0 + (s + kAhead) / NCT), (s + kAhead) % NCT, xb[(s + kAhead) % kSlots]);
          __builtin_amdgcn_sched_barrier(0);
          if (ct == 0) {
            pacc[0] = f32x16{};
            pacc[1] = f32x16{};
          }
#pragma unroll
          for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int t = 0; t < 2; ++t) {
              const u32x4(&xq)[P] = xb[s % kSlots][q];
              const u32x4(&gq)[P] = ghp[t][ct][q];
              if constexpr (!BF) {
                pacc[t] = mfma16<BF>(xq[1], gq[0], pacc[t]);
                pacc[t] = mfma16<BF>(xq[0], gq[1], pacc[t]);
              }
              pacc[t] = mfma16<BF>(xq[0], gq[0], pacc[t]);
            }
          __builtin_amdgcn_sched_barrier(0);
          if (ct + 1 == NCT && e < n) {
            const float sc = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(sc_l), e));
#pragma unroll
            for (int t = 0; t < 2; ++t) {
              float part = 0.f;
#pragma unroll
              for (int qq = 0; qq < 4; ++qq) {
                const f32x4 av = sAl[((kt * RT + rtw[t]) * 4 + qq) * kWave + lane];
#pragma unroll
                for (int i = 0; i < 4; ++i) part += av[i] * pacc[t][4 * qq + i];
              }
              part += __shfl_xor(part, 32);
              if (h == 0 && keep[t])
                dgb[(e % kChunk) * Rs + rtw[t] * kTile + l32] = part * (sc * gh_unscale[t]);
            }
          }
        }
        // a chunk is whole: its k tiles' parts added and stored (the other
        // buffer's were, before this barrier)
        if ((e0 + 2) % kChunk == 0 || e0 + 2 >= n) {
          lds_barrier();
          const int c0 = e0 / kChunk * kChunk, m = min(kChunk, n - c0);
          const float* in = sDG + ((e0 / kChunk) & 1) * MT * kChunk * Rs;
          for (int i = tid; i < m * Rp; i += blockDim.x) {
            const int e = i / Rp, r = i - e * Rp;
            float v = in[e * Rs + r];
#pragma unroll
            for (int k2 = 1; k2 < MT; ++k2) v += in[(k2 * kChunk + e) * Rs + r];
            if (r < R) a.dg[size_t(a.perm[cb + c0 + e]) * R + r] = v;
          }
        }
      }
    }
  }
}

template <int MT, int RT, int NCT, bool BF>
hipError_t launch_k(const BwdDstArgs& a, hipStream_t s) {
  const size_t lds = size_t(dg_smem(RT, MT, a.d, a.C, gh_floats(MT, RT, NCT, BF ? 1 : 2)).floats) * 4;
  if (lds > 160 * 1024) return hipErrorInvalidValue;
  auto k = k_bwd_dg_direct<MT, RT, NCT, BF>;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize,
                                     int(lds));
  if (e != hipSuccess) return e;
  // as many workgroups as the device holds (by LDS, and two waves per SIMD)
  const int by_lds = int(160 * 1024 / lds), by_waves = (NCT == 8 ? 4 : 8) / direct_waves(MT, RT);
  const int per_cu = max(1, min(by_lds, by_waves)), most = per_cu * device_cus();
  k<<<dim3(min(a.n_seg, most)), dim3(direct_waves(MT, RT) * kWave), lds, s>>>(a);
  return hipGetLastError();
}

template <int MT, bool BF>
hipError_t launch_mt(const BwdDstArgs& a, hipStream_t s) {
  const int rt = (a.R + kTile - 1) / kTile;
  const int NC = bwd_direct_cpad(a.C) / kTile;
#define TDN_BWD_CASE(RTV)                                   \
  case RTV:                                                 \
    if (NC == 2) return launch_k<MT, RTV, 2, BF>(a, s);     \
    if (NC == 4) return launch_k<MT, RTV, 4, BF>(a, s);     \
    return launch_k<MT, RTV, 8, BF>(a, s);
  switch (rt) {
    TDN_BWD_CASE(1)
    TDN_BWD_CASE(2)
    TDN_BWD_CASE(3)
    TDN_BWD_CASE(4)
    TDN_BWD_CASE(5)
    TDN_BWD_CASE(6)
    TDN_BWD_CASE(7)
    TDN_BWD_CASE(8)
    default: return hipErrorInvalidValue;
  }
#undef TDN_BWD_CASE
}

}  // namespace bwd_detail

}  // namespace tdn
