// bca_block_kernels.hpp -- fused block-circulant layer kernels (Sec. 3.3, Eqs. (4)-(5)) whose
// per-bin block products run on the matrix cores, for layers of many blocks or rectangular
// ones (p = 128 ... 1024, up to 16 x 16 blocks).
//
// Per bin k the layer is a small complex matrix product over the tokens of a tile:
//   Y[k] = C[k] X[k],   dX[k] = C[k]^H G[k],   dC[k] += G[k] X[k]^H.
// v_mfma_f32_4x4x1_16b_f32 multiplies sixteen independent 4x1 by 1x4 pairs in float32: with
// one block of the instruction per bin, four rows (output blocks), four columns (tokens, or
// input blocks for dC) and one block or token per step, nothing of it is padding when the
// block counts are multiples of four.  It has the exact float32 products and sums of the VALU
// form at twice its rate, and leaves the VALU to the transforms, which bound these kernels.
// The lane (bin l/4, column l%4) reads its operands straight from the spectra in LDS, and
// four of its results per lane are the float2 slots it writes back.
//
// Slot 0 holds the real bins Y_0 and Y_{p/2}: its products are elementwise, which the lanes
// of bin 0 get from the same instructions by taking other operands (zero for the cross terms).
#pragma once

#include "bca_kernels.hpp"

namespace rdfft {

typedef float f32x4_t __attribute__((ext_vector_type(4)));

// D[row r][col] += A[row] B[col] for each of the 16 blocks of four lanes: lane l holds row l%4
// of A, column l%4 of B, and rows 0..3 of column l%4 of D, all of block l/4
__device__ __forceinline__ f32x4_t mfma_4x4(float a, float b, f32x4_t d) {
  return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, d, 0, 0, 0);
}

// whether block m exists in every layer of G groups of four (1 group: 1..4 blocks, 2: 5..8,
// 4: 9..16); the other blocks are tested, and take part as zeros when absent
constexpr bool sure(int m, int G) { return m < (G == 1 ? 1 : G == 2 ? 5 : 9); }

template <int LOGN>
struct BcaBlock {
  using P = RowPlan<LOGN>;
  static constexpr int N = P::N, TPR = P::TPR;
  static constexpr int NB = N / 16;  // 16-bin groups
  static_assert(N >= 64 && TPR <= 64, "rows of one wavefront, whole bin groups");
  // Region of one spectrum, a stride of 8 (mod 16) float2: the four rows (blocks) that a
  // wave reads side by side, 8 consecutive bins each per 32 lanes, then lie on all 64 banks once
  static constexpr int MIN_REG = P::LDS_F2 > lds_padded_size(N) ? P::LDS_F2 : lds_padded_size(N);
  static constexpr int REG = MIN_REG + (24 - MIN_REG % 16) % 16;
};
// ... and the same for the stride between a tile's tokens (float2)
template <int LOGN>
__host__ __device__ constexpr int block_token_stride(int regions) {
  const int s = regions * BcaBlock<LOGN>::REG;
  return s + (24 - s % 16) % 16;
}

// Forward of one tile of TT tokens per turn of a persistent workgroup; X_j in LDS, Y_i over
// it (max(q, kb) regions per token).  KG: groups of four input blocks, 4*KG >= kb.
template <int LOGN, class St, int KG, int WG>
__global__ void __launch_bounds__(WG) __attribute__((amdgpu_waves_per_eu(4)))
bca_forward_block_kernel(const ElemOf<St>* x, const ElemOf<St>* __restrict__ c, ElemOf<St>* y, int64_t tokens, int q,
                         int kb, int TT, int TS, int64_t ntiles, const float2* __restrict__ tw) {
  using B = BcaBlock<LOGN>;
  using In = typename St::In;
  using Out = typename St::Out;
  constexpr int N = B::N, TPR = B::TPR, REG = B::REG, NB = B::NB, NG = WG / TPR, NW = WG / 64, RPW = 64 / TPR;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // (uniform: matrix instructions ignore the lane mask)
  const int grp = tid / TPR, t = tid - grp * TPR;
  float2* const xs = bca_lds;                  // TT tokens of TS float2
  float2* const dummy = bca_lds + (size_t)TT * TS;
  const In cin{c};
  const int TG = (TT + 3) / 4, QG = (q + 3) / 4;
  const int U = NB * TG;                       // units: 16 bins of 4 tokens
  const int HS = U < NW ? NW / U : 1;          // waves that share a unit, by output groups
  const int b = lane >> 2, n = lane & 3;

  for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const int64_t tok0 = tile * TT;
    const int nvalid = (int)(tokens - tok0 < TT ? tokens - tok0 : TT);

    const int nx = TT * kb;
    for (int s0 = 0; s0 < nx; s0 += NG) {
      if (s0 + wave * RPW >= nx) continue;  // rows synchronise at wave level: an idle wave leaves
      const int s = s0 + grp;
      const bool valid = s < nx;
      const int tt = valid ? s / kb : 0, j = valid ? s - tt * kb : 0;
      const bool act = valid && tt < nvalid;
      float2* reg = valid ? xs + tt * TS + j * REG : dummy;
      const In src{x + ((act ? tok0 + tt : 0) * kb + j) * (int64_t)N};
      row_forward<LOGN, true>(t, act, src, LdsSpectrum{reg}, reg, tw);
    }
    // Y_i[k] = sum_j C_ij[k] X_j[k]: rows i, columns tokens, one input block per step.  Up to 8
    // input blocks, the C rows of the next output group are in flight while one is computed,
    // the first group's across the barrier (more blocks do not leave the registers for that).
    constexpr bool AHEAD = KG <= 2;
    int u = wave / HS;
    const int h = wave % HS;
    typename In::raw_t raw[4 * KG];
    auto load_c = [&](int unit, int ig) {
      const int i = 4 * ig + n < q ? 4 * ig + n : q - 1;  // (rows past q repeat the last)
      const int ci = i * kb * N + 16 * (unit % NB) + b;
      static_for<4 * KG>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        raw[j] = cin.load_raw(ci + (sure(j, KG) || j < kb ? j : 0) * N);
      });
    };
    if constexpr (AHEAD) load_c(u, h);
    __syncthreads();
    for (int u0 = 0; u0 < U; u0 += NW, u += NW) {
      const bool busy = u < U;
      const int g = u % NB, tg = u / NB;
      const int bin = 16 * g + b;
      const int tok = 4 * tg + n < TT ? 4 * tg + n : TT - 1;  // (columns past the tile repeat its last)
      float2* const base = xs + (busy ? tok : 0) * TS + lds_pad(bin);
      float2 X[4 * KG];
      static_for<4 * KG>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        X[j] = make_float2(0.f, 0.f);
        if (sure(j, KG) || j < kb) X[j] = base[j * REG];
      });
      // waves that share a unit read all of its X before any of them writes Y over it
      if (HS > 1) __syncthreads();
      if (!busy) continue;
      auto outputs = [&](auto s0c) {
        constexpr bool S0 = decltype(s0c)::value;
        for (int ig = h; ig < QG; ig += HS) {
          if constexpr (!AHEAD) load_c(u, ig);
          typename In::raw_t cur[4 * KG];
          static_for<4 * KG>([&](auto jc) { cur[decltype(jc)::value] = raw[decltype(jc)::value]; });
          if constexpr (AHEAD) {
            if (ig + HS < QG) load_c(u, ig + HS);
            else if (u + NW < U) load_c(u + NW, h);
          }
          f32x4_t rr = {0.f, 0.f, 0.f, 0.f}, ii = rr, ir = rr, ri = rr;
          static_for<4 * KG>([&](auto jc) {
            constexpr int j = decltype(jc)::value;
            float2 cv = In::widen(cur[j]);
            if (!sure(j, KG) && j >= kb) cv = make_float2(0.f, 0.f);
            const float im = S0 && b == 0 ? 0.f : cv.y;  // cross terms: none in slot 0
            const float di = S0 && b == 0 ? cv.y : cv.x;
            rr = mfma_4x4(cv.x, X[j].x, rr);
            ii = mfma_4x4(im, X[j].y, ii);
            ir = mfma_4x4(im, X[j].x, ir);
            ri = mfma_4x4(di, X[j].y, ri);
          });
          const f32x4_t re = rr - ii, im = ir + ri;
          static_for<4>([&](auto rc) {
            constexpr int r = decltype(rc)::value;
            if (4 * ig + r < q) base[(4 * ig + r) * REG] = make_float2(re[r], im[r]);
          });
        }
      };
      if (g == 0) outputs(std::true_type{});
      else outputs(std::false_type{});
    }
    __syncthreads();

    const int ny = TT * q;
    for (int s0 = 0; s0 < ny; s0 += NG) {
      if (s0 + wave * RPW >= ny) continue;
      const int s = s0 + grp;
      const bool valid = s < ny;
      const int tt = valid ? s / q : 0, i = valid ? s - tt * q : 0;
      const bool act = valid && tt < nvalid;
      float2* reg = valid ? xs + tt * TS + i * REG : dummy;
      const Out dst{y + ((act ? tok0 + tt : 0) * q + i) * (int64_t)N};
      row_inverse<LOGN, true>(t, act, LdsSpectrum{reg}, dst, reg, tw);
    }
    __syncthreads();
  }
}

constexpr int gcd2(int a, int b) { return b == 0 ? a : gcd2(b, a % b); }

// Backward split: a wave owns the 16-bin groups wave + bt*NW (BT of them), or HS waves share
// one group and split its 4x4 tiles of dC (SI by output groups, SJ by input groups).
template <int LOGN, int QG, int KG, int WG>
struct BcaBlockBwd {
  static constexpr int NW = WG / 64, NB = BcaBlock<LOGN>::NB;
  static constexpr int HS = NB < NW ? NW / NB : 1;
  static constexpr int BT = NB < NW ? 1 : NB / NW;
  static constexpr int SI = gcd2(QG, HS), SJ = gcd2(KG, HS / SI);
  static constexpr int IGW = QG / SI, JGW = KG / SJ;
  static constexpr int ACC = BT * IGW * JGW * 8;  // dC registers per lane
};

// Backward of one tile per turn: X_j and G_i in LDS (kb + q regions per token), dC_ij in
// registers for all of the workgroup's tiles, dX_j over X_j.  The partial sums leave at the
// end to `stage` (chunk_rows rows of dC into the gy rows of each of the workgroup's first
// tiles, which it alone has read) or, stage == nullptr, by float32 atomics into dc.
template <int LOGN, class St, int QG, int KG, int WG>
__global__ void __launch_bounds__(WG)
bca_backward_block_kernel(const ElemOf<St>* __restrict__ x, const ElemOf<St>* __restrict__ c, const ElemOf<St>* gy,
                          ElemOf<St>* dx, float* __restrict__ dc, int64_t tokens, int q, int kb, int TT, int TS,
                          int64_t ntiles, float2* stage, int64_t tile_f2, int chunk_rows, const float2* __restrict__ tw) {
  using B = BcaBlock<LOGN>;
  using S = BcaBlockBwd<LOGN, QG, KG, WG>;
  using In = typename St::In;
  using Out = typename St::Out;
  constexpr int N = B::N, TPR = B::TPR, REG = B::REG, NB = B::NB, NG = WG / TPR, NW = S::NW, HS = S::HS, BT = S::BT;
  constexpr int IGW = S::IGW, JGW = S::JGW, RPW = 64 / TPR;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // (uniform: matrix instructions ignore the lane mask)
  const int grp = tid / TPR, t = tid - grp * TPR;
  float2* const xs = bca_lds;  // per token: kb regions X, then dX; q regions G
  float2* const dummy = bca_lds + (size_t)TT * TS;
  const In cin{c};
  const int b = lane >> 2, n = lane & 3;
  const int g0 = wave / HS, h = wave % HS;       // first bin group, share of it
  const int hi = h % S::SI, hj = (h / S::SI) % S::SJ;
  const bool dc_busy = h < S::SI * S::SJ;
  if (stage != nullptr) {  // the second stage, later on the stream, adds into dc
    for (int64_t e = (int64_t)blockIdx.x * WG + tid; e < 2 * (int64_t)q * kb * N; e += (int64_t)gridDim.x * WG)
      dc[e] = 0.f;
  }
  f32x4_t dre[BT][IGW][JGW], dim_[BT][IGW][JGW];
  static_for<BT>([&](auto bc) {
    static_for<IGW>([&](auto ic) {
      static_for<JGW>([&](auto jc) {
        dre[decltype(bc)::value][decltype(ic)::value][decltype(jc)::value] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        dim_[decltype(bc)::value][decltype(ic)::value][decltype(jc)::value] = f32x4_t{0.f, 0.f, 0.f, 0.f};
      });
    });
  });

  for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const int64_t tok0 = tile * TT;
    const int nvalid = (int)(tokens - tok0 < TT ? tokens - tok0 : TT);

    const int per = kb + q, ns = TT * per;
#pragma unroll 1
    for (int s0 = 0; s0 < ns; s0 += NG) {
      if (s0 + wave * RPW >= ns) continue;  // rows synchronise at wave level: an idle wave leaves
      const int s = s0 + grp;
      const bool valid = s < ns;
      const int tt = valid ? s / per : 0, m = valid ? s - tt * per : 0;
      const bool act = valid && tt < nvalid;
      float2* reg = valid ? xs + tt * TS + m * REG : dummy;
      const int64_t tok = act ? tok0 + tt : 0;
      const ElemOf<St>* srcp = m < kb ? x + (tok * kb + m) * (int64_t)N : gy + (tok * q + (m - kb)) * (int64_t)N;
      row_forward<LOGN, true>(t, act, In{srcp}, LdsSpectrum{reg}, reg, reread(tw));
    }
    __syncthreads();

    // dC_ij[k] += sum_t conj(X_tj[k]) G_ti[k]: rows i, columns j, one token per step
    if (dc_busy) {
      static_for<BT>([&](auto bc) {
        constexpr int bt = decltype(bc)::value;
        const int bin = 16 * (g0 + bt * NW) + b;
        const bool z = bin == 0;
        const float2* gp[IGW];
        const float2* xp[JGW];
        static_for<IGW>([&](auto ic) {
          constexpr int ii = decltype(ic)::value;
          const int i = 4 * (hi + ii * S::SI) + n;
          gp[ii] = xs + (kb + (i < q ? i : q - 1)) * REG + lds_pad(bin);
        });
        static_for<JGW>([&](auto jc) {
          constexpr int jj = decltype(jc)::value;
          const int j = 4 * (hj + jj * S::SJ) + n;
          xp[jj] = xs + (j < kb ? j : kb - 1) * REG + lds_pad(bin);
        });
#pragma unroll 2
        for (int tt = 0; tt < nvalid; ++tt) {
          float2 G[IGW], X[JGW];
          float gi[IGW], gn[IGW], xr[JGW];
          static_for<IGW>([&](auto ic) { G[decltype(ic)::value] = gp[decltype(ic)::value][tt * TS]; });
          static_for<JGW>([&](auto jc) { X[decltype(jc)::value] = xp[decltype(jc)::value][tt * TS]; });
          // slot 0: G.x X.x and G.y X.y alone
          static_for<IGW>([&](auto ic) {
            constexpr int ii = decltype(ic)::value;
            gi[ii] = z ? 0.f : G[ii].y;
            gn[ii] = z ? 0.f : -G[ii].x;
          });
          static_for<JGW>([&](auto jc) { xr[decltype(jc)::value] = z ? X[decltype(jc)::value].y : X[decltype(jc)::value].x; });
          static_for<IGW>([&](auto ic) {
            constexpr int ii = decltype(ic)::value;
            static_for<JGW>([&](auto jc) {
              constexpr int jj = decltype(jc)::value;
              dre[bt][ii][jj] = mfma_4x4(G[ii].x, X[jj].x, dre[bt][ii][jj]);
              dim_[bt][ii][jj] = mfma_4x4(G[ii].y, xr[jj], dim_[bt][ii][jj]);
            });
          });
          static_for<IGW>([&](auto ic) {
            constexpr int ii = decltype(ic)::value;
            static_for<JGW>([&](auto jc) {
              constexpr int jj = decltype(jc)::value;
              dre[bt][ii][jj] = mfma_4x4(gi[ii], X[jj].y, dre[bt][ii][jj]);
              dim_[bt][ii][jj] = mfma_4x4(gn[ii], X[jj].y, dim_[bt][ii][jj]);
            });
          });
        }
      });
    }
    // waves that share a bin group read all of its X before any of them writes dX over it
    if constexpr (HS > 1) __syncthreads();

    // dX_j[k] = sum_i conj(C_ij[k]) G_i[k]: rows j, columns tokens, one output block per step
    const int TG = (TT + 3) / 4;
#pragma unroll 1
    for (int bt = 0; bt < BT; ++bt) {
      const int g = g0 + bt * NW, bin = 16 * g + b;
      auto grad_x = [&](auto s0c) {
        constexpr bool S0 = decltype(s0c)::value;
#pragma unroll 1
        for (int jg = h; jg < (kb + 3) / 4; jg += HS) {
          const int j = 4 * jg + n < kb ? 4 * jg + n : kb - 1;  // (rows past kb repeat the last)
          const int ci = j * N + bin;
          typename In::raw_t raw[4 * QG];
          static_for<4 * QG>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            raw[i] = cin.load_raw(ci + (sure(i, QG) || i < q ? i : 0) * kb * N);
          });
#pragma unroll 1
          for (int tg = 0; tg < TG; ++tg) {
            const int tok = 4 * tg + n < TT ? 4 * tg + n : TT - 1;
            float2* const base = xs + tok * TS + lds_pad(bin);
            f32x4_t rr = {0.f, 0.f, 0.f, 0.f}, ii = rr, ri = rr, ir = rr;
            static_for<4 * QG>([&](auto ic) {
              constexpr int i = decltype(ic)::value;
              float2 gv = make_float2(0.f, 0.f), cv = In::widen(raw[i]);
              if (sure(i, QG) || i < q) gv = base[(kb + i) * REG];
              else cv = gv;
              const float im = S0 && b == 0 ? 0.f : cv.y;
              const float di = S0 && b == 0 ? cv.y : cv.x;
              rr = mfma_4x4(cv.x, gv.x, rr);
              ii = mfma_4x4(im, gv.y, ii);
              ri = mfma_4x4(di, gv.y, ri);
              ir = mfma_4x4(im, gv.x, ir);
            });
            const f32x4_t re = rr + ii, im = ri - ir;
            static_for<4>([&](auto rc) {
              constexpr int r = decltype(rc)::value;
              if (4 * jg + r < kb) base[(4 * jg + r) * REG] = make_float2(re[r], im[r]);
            });
          }
        }
      };
      if (g == 0) grad_x(std::true_type{});
      else grad_x(std::false_type{});
    }
    __syncthreads();

    const int nx = TT * kb;
#pragma unroll 1
    for (int s0 = 0; s0 < nx; s0 += NG) {
      if (s0 + wave * RPW >= nx) continue;
      const int s = s0 + grp;
      const bool valid = s < nx;
      const int tt = valid ? s / kb : 0, j = valid ? s - tt * kb : 0;
      const bool act = valid && tt < nvalid;
      float2* reg = valid ? xs + tt * TS + j * REG : dummy;
      const Out dst{dx + ((act ? tok0 + tt : 0) * kb + j) * (int64_t)N};
      row_inverse<LOGN, true>(t, act, LdsSpectrum{reg}, dst, reg, reread(tw));
    }
    __syncthreads();
  }

  // visit(ij, v): row ij = i*kb + j of dC, slot 16*(g0 + bt*NW) + b (bin) of it
  auto each = [&](auto&& visit) {
    static_for<BT>([&](auto bc) {
      constexpr int bt = decltype(bc)::value;
      const int bin = 16 * (g0 + bt * NW) + b;
      static_for<IGW>([&](auto ic) {
        constexpr int ii = decltype(ic)::value;
        static_for<JGW>([&](auto jc) {
          constexpr int jj = decltype(jc)::value;
          const int j = 4 * (hj + jj * S::SJ) + n;
          static_for<4>([&](auto rc) {
            constexpr int r = decltype(rc)::value;
            const int i = 4 * (hi + ii * S::SI) + r;
            if (i < q && j < kb) visit(i * kb + j, bin, make_float2(dre[bt][ii][jj][r], dim_[bt][ii][jj][r]));
          });
        });
      });
    });
  };
  if (stage != nullptr) {
    if (!dc_busy) return;
    const float inv_rows = 1.0f / (float)chunk_rows;
    each([&](int ij, int bin, float2 v) {
      const int ch = (int)(((float)ij + 0.5f) * inv_rows);  // ij / chunk_rows, exact: ij < 256
      stage[((int64_t)blockIdx.x + (int64_t)ch * gridDim.x) * tile_f2 + (ij - ch * chunk_rows) * N + bin] = v;
    });
    return;
  }
  // by atomics: as many rows at a time as the spectra's LDS holds (the last tile is done with it)
  const int at_once = (TT * TS + REG) / N;
  for (int r0 = 0; r0 < q * kb; r0 += at_once) {
    const int nr = q * kb - r0 < at_once ? q * kb - r0 : at_once;
    if (dc_busy)
      each([&](int ij, int bin, float2 v) {
        if (ij >= r0 && ij < r0 + nr) bca_lds[(ij - r0) * N + bin] = v;
      });
    __syncthreads();
    atomic_add_rotated<WG, 1, 1>(dc + (int64_t)r0 * 2 * N, reinterpret_cast<const float*>(bca_lds), nr * 2 * N);
    __syncthreads();
  }
}

// ----------------------------------------------------------------------------------
// host side
constexpr int kBlockMinLogN = 6, kBlockMaxLogN = 9;  // p = 128 ... 1024
constexpr int kBlockFwdWG = 512;
constexpr int kBlockMaxBlocks = 16;

// group counts the kernels are built for: 1, 2 or 4 groups of four blocks
constexpr int block_groups_index(int blocks) { return blocks <= 4 ? 0 : blocks <= 8 ? 1 : 2; }

template <int LOGN, int QG, int KG>
constexpr int block_bwd_wg() {
  return BcaBlockBwd<LOGN, QG, KG, 1024>::ACC <= 48 ? 1024 : 512;
}
// whether LDS holds four tokens of `regions` spectra and a spare region
template <int LOGN>
constexpr bool block_tile_fits(int regions) {
  return (4 * block_token_stride<LOGN>(regions) + BcaBlock<LOGN>::REG) * (int)sizeof(float2) <= kLdsLimit;
}
constexpr int fewest_blocks(int G) { return G == 1 ? 1 : G == 2 ? 5 : 9; }  // of a layer of G groups

// built when the dC registers leave room for the transforms (128 or 256 registers per lane), and LDS for a
// tile of the fewest blocks
template <int LOGN, int QG, int KG>
constexpr bool block_bwd_fits() {
  constexpr int wg = block_bwd_wg<LOGN, QG, KG>();
  return BcaBlockBwd<LOGN, QG, KG, wg>::ACC <= (wg == 1024 ? 48 : 128) &&
         block_tile_fits<LOGN>(fewest_blocks(QG) + fewest_blocks(KG));
}

// Tokens per tile of the forward: a multiple of four up to `most` within `budget` bytes that still
// gives every CU `per_cu` tiles, or fewer than four when the batch is too short to give every CU four; 0
// when the tile does not fit.  (One tile per CU, of up to four tokens, comes before a second one: 1021
// tokens of 12 x 12 blocks of 256, float32, as tiles of two took 29 us, of four 20.)
template <int LOGN>
static int block_tile_tokens(int regions, int64_t tokens, int num_cu, int per_cu, int most, int budget) {
  const int64_t ts = (int64_t)block_token_stride<LOGN>(regions) * 8, spare = BcaBlock<LOGN>::REG * 8;
  int tt = most;
  while (tt > 4 && (tt * ts + spare > budget || (int64_t)tt * num_cu * per_cu > tokens)) tt -= 4;
  if (tt * ts + spare > budget) return 0;
  const int64_t share = std::max<int64_t>(1, (tokens + num_cu - 1) / num_cu);
  return (int)std::min<int64_t>(tt, share);
}

template <int LOGN, class St, int KG>
static hipError_t fwd_block_impl(const BcaArgs& a, const float2* tw, hipStream_t stream, int num_cu) {
  constexpr int WG = kBlockFwdWG;
  const int regions = std::max(a.q, a.kb);
  int TT = block_tile_tokens<LOGN>(regions, a.tokens, num_cu, 2, 16, kLdsLimit / 2);
  if (TT == 0) TT = block_tile_tokens<LOGN>(regions, a.tokens, num_cu, 1, 4, kLdsLimit);
  if (TT == 0) return hipErrorInvalidValue;
  const int TS = block_token_stride<LOGN>(regions);
  const size_t lds = ((size_t)TT * TS + BcaBlock<LOGN>::REG) * sizeof(float2);
  static const hipError_t attr = set_lds_limit(bca_forward_block_kernel<LOGN, St, KG, WG>);
  if (attr != hipSuccess) return attr;
  const int64_t tiles = (a.tokens + TT - 1) / TT;
  const int per_cu = std::max(1, std::min<int>(kLdsLimit / (int)lds, 2048 / WG));
  const int64_t grid = std::min<int64_t>(tiles, (int64_t)num_cu * per_cu);
  hipLaunchKernelGGL((bca_forward_block_kernel<LOGN, St, KG, WG>), dim3((unsigned)grid), dim3(WG), lds, stream,
                     static_cast<const ElemOf<St>*>(a.x), static_cast<const ElemOf<St>*>(a.c),
                     static_cast<ElemOf<St>*>(a.y), a.tokens, a.q, a.kb, TT, TS, tiles, tw);
  return hipGetLastError();
}

constexpr int kBlockStageMinGrid = 8;
constexpr int kBlockFewBlocks = 6;

// How the backward runs a batch: tiles of TT tokens
struct BlockBwdRun {
  int TT;
  int64_t tiles, grid, tile_f2, chain;
  int chunk_rows;
  bool staged, repeatable;  // repeatable: at most two atomic additions to a value of dc
  bool general;             // the general kernel is the faster one
};
template <int LOGN, class St>
static BlockBwdRun block_bwd_run(const BcaArgs& a, int num_cu, int TT) {
  constexpr int N = BcaBlock<LOGN>::N;
  BlockBwdRun r{};
  r.TT = TT;
  r.tiles = (a.tokens + TT - 1) / TT;
  r.grid = std::min<int64_t>(r.tiles, num_cu);
  // two-stage dC sum in consumed gy rows (dx apart from gy), as in the square-layer kernels
  const int64_t blocks = (int64_t)a.q * a.kb, full = a.tokens / TT;
  r.tile_f2 = (int64_t)TT * a.q * N * (int64_t)sizeof(ElemOf<St>) / (int64_t)sizeof(float2);
  r.chunk_rows = (int)std::max<int64_t>(1, std::min<int64_t>(blocks, r.tile_f2 / N));
  const int64_t chunks = (blocks + r.chunk_rows - 1) / r.chunk_rows;
  // (staged only when every workgroup has whole tiles enough: fewer workgroups that all do cost more
  // than the atomics, 42 us against 40 us for 16 x 4 blocks of 256 over 2045 tokens; and for enough of
  // them: with two, 8 tokens of 1 x 2 blocks of 1024, 16.0 us against 14.0.  From eight on it is the faster
  // one in nearly every layer: 128 tokens 0.78, 4096 tokens 0.75 of the time by atomics)
  r.staged = a.dx != a.y && !a.keep_gy && r.tile_f2 >= N && r.grid >= kBlockStageMinGrid && chunks * r.grid <= full;
  r.chain = dc_chain(a.tokens, r.grid, 1, r.staged);
  r.repeatable = r.grid <= (r.staged ? 2 * kReduceGroup : 2);
  return r;
}

// Tokens of the backward's tile: a multiple of four (or a batch of fewer).  At least a CU's share, up to what
// fills the row groups of the inverse round (one block row of 128 and two columns, 8192 tokens: 39 us with
// four, 18 us); and more, as far as LDS holds them, until dC's sum has no more additions in a row, and
// repeats, as in the general kernel with its tiles.
template <int LOGN, class St, int WG>
static BlockBwdRun block_bwd_pick(const BcaArgs& a, int num_cu) {
  using B = BcaBlock<LOGN>;
  const int64_t ts = (int64_t)block_token_stride<LOGN>(a.q + a.kb) * 8, spare = B::REG * 8;
  const int most = (int)std::min<int64_t>(64, (kLdsLimit - spare) / ts / 4 * 4);
  if (a.tokens < 4) return block_bwd_run<LOGN, St>(a, num_cu, (int)a.tokens);
  constexpr int gwg = BcaPlan<LOGN>::BWD_WG;
  int ia = a.q, jb = a.kb;
  if (!dc_whole(LOGN, gwg, a.q, a.kb, num_cu)) dc_chunk(LOGN, a.q, a.kb, &ia, &jb);
  const BwdTiles general = bwd_tiles(LOGN, gwg, ia, jb, a.tokens, num_cu, true);
  const int64_t chain = dc_chain(a.tokens, std::max<int64_t>(1, general.grid), 1, false);
  const int fill = (WG / B::TPR + a.kb - 1) / a.kb;
  const int64_t share = std::min<int64_t>(fill, (a.tokens + num_cu - 1) / num_cu);
  int TT = (int)std::min<int64_t>(most, (share + 3) / 4 * 4);
  BlockBwdRun r = block_bwd_run<LOGN, St>(a, num_cu, TT);
  while (TT < most && TT < a.tokens && (r.chain > chain || (general.grid <= 2 && !r.repeatable)))
    r = block_bwd_run<LOGN, St>(a, num_cu, TT += 4);
  // Few blocks, whose dC sums are four of the sixteen waves' work here: with tiles near the general
  // kernel's and nothing staged, that one is ahead (1 x 2 blocks of 128, 128 tokens, gy kept: 16.9 us : 27.3)
  r.general = !r.staged && a.q * a.kb <= kBlockFewBlocks && 4 * r.TT >= 3 * general.TT;
  return r;
}

template <int LOGN, class St, int QG, int KG>
static hipError_t bwd_block_impl(const BcaArgs& a, const float2* tw, hipStream_t stream, int num_cu) {
  constexpr int WG = block_bwd_wg<LOGN, QG, KG>();
  constexpr int N = BcaBlock<LOGN>::N;
  const BlockBwdRun r = block_bwd_pick<LOGN, St, WG>(a, num_cu);
  if (r.general) return hipErrorNotSupported;  // nothing launched: the caller runs the general kernel
  const int TS = block_token_stride<LOGN>(a.q + a.kb);
  const size_t lds = ((size_t)r.TT * TS + BcaBlock<LOGN>::REG) * sizeof(float2);
  if (lds > (size_t)kLdsLimit) return hipErrorInvalidValue;
  static const hipError_t attr = set_lds_limit(bca_backward_block_kernel<LOGN, St, QG, KG, WG>);
  if (attr != hipSuccess) return attr;
  float2* const stage = r.staged ? static_cast<float2*>(a.y) : nullptr;
  if (!r.staged) {
    const hipError_t ez = launch_fill_zero(a.dc, 2 * (int64_t)a.q * a.kb * N, stream);
    if (ez != hipSuccess) return ez;
  }
  hipLaunchKernelGGL((bca_backward_block_kernel<LOGN, St, QG, KG, WG>), dim3((unsigned)r.grid), dim3(WG), lds, stream,
                     static_cast<const ElemOf<St>*>(a.x), static_cast<const ElemOf<St>*>(a.c),
                     static_cast<const ElemOf<St>*>(a.y), static_cast<ElemOf<St>*>(a.dx), a.dc, a.tokens, a.q, a.kb,
                     r.TT, TS, r.tiles, stage, r.tile_f2, r.chunk_rows, tw);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (r.staged)
    return launch_dc_finish(stage, a.dc, a.q * a.kb, LOGN, r.chunk_rows * N, (int)r.grid, r.tile_f2, tw, stream);
  return launch_rdfft_rows(a.dc, (int64_t)a.q * a.kb, LOGN, kStorageF32, true, tw, stream, num_cu);
}

template <int LOGN, class St, int QG, int KG>
static constexpr BcaBwdFn block_bwd_entry() {
  if constexpr (block_bwd_fits<LOGN, QG, KG>()) return &bwd_block_impl<LOGN, St, QG, KG>;
  else return nullptr;
}
template <int LOGN, class St>
static constexpr std::array<std::array<BcaBwdFn, 3>, 3> block_bwd_entries() {
  return {{{block_bwd_entry<LOGN, St, 1, 1>(), block_bwd_entry<LOGN, St, 1, 2>(), block_bwd_entry<LOGN, St, 1, 4>()},
           {block_bwd_entry<LOGN, St, 2, 1>(), block_bwd_entry<LOGN, St, 2, 2>(), block_bwd_entry<LOGN, St, 2, 4>()},
           {block_bwd_entry<LOGN, St, 4, 1>(), block_bwd_entry<LOGN, St, 4, 2>(), block_bwd_entry<LOGN, St, 4, 4>()}}};
}
template <int LOGN, class St, int KG>
static constexpr BcaBwdFn block_fwd_entry() {
  if constexpr (block_tile_fits<LOGN>(fewest_blocks(KG))) return &fwd_block_impl<LOGN, St, KG>;
  else return nullptr;
}
template <int LOGN, class St>
static constexpr std::array<BcaBwdFn, 3> block_fwd_entries() {
  return {block_fwd_entry<LOGN, St, 1>(), block_fwd_entry<LOGN, St, 2>(), block_fwd_entry<LOGN, St, 4>()};
}

// [logn - kBlockMinLogN][input groups] and [logn - kBlockMinLogN][output groups][input groups]
constexpr int kBlockPlans = kBlockMaxLogN - kBlockMinLogN + 1;
struct BcaBlockTables {
  std::array<std::array<BcaBwdFn, 3>, kBlockPlans> fwd;
  std::array<std::array<std::array<BcaBwdFn, 3>, 3>, kBlockPlans> bwd;
};
template <class St, int... L>
static BcaBlockTables make_block_tables(std::integer_sequence<int, L...>) {
  return {{block_fwd_entries<L + kBlockMinLogN, St>()...}, {block_bwd_entries<L + kBlockMinLogN, St>()...}};
}

// bytes of LDS that `tokens` tokens of `regions` spectra and a spare region take
static int64_t block_lds_bytes(int logn, int regions, int tokens) {
  switch (logn) {
    case 6: return ((int64_t)tokens * block_token_stride<6>(regions) + BcaBlock<6>::REG) * 8;
    case 7: return ((int64_t)tokens * block_token_stride<7>(regions) + BcaBlock<7>::REG) * 8;
    case 8: return ((int64_t)tokens * block_token_stride<8>(regions) + BcaBlock<8>::REG) * 8;
    case 9: return ((int64_t)tokens * block_token_stride<9>(regions) + BcaBlock<9>::REG) * 8;
    default: return INT64_MAX;
  }
}

BcaBlockTables bca_block_tables_f32();
BcaBlockTables bca_block_tables_bf16();
BcaBlockTables bca_block_tables_f16();

}  // namespace rdfft
