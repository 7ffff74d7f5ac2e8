// HIP kernels for decentralized uplink detection and downlink precoding on gfx950.
//
// Method: Li et al., "Decentralized Baseband Processing for Massive MU-MIMO
// Systems" (arXiv:1702.04458).  Algorithm 1 (decentralized ADMM detection,
// U x U branch, eq. StepE1variant1), Algorithm 2 (decentralized CG detection,
// eqs. CGiteration / CGdecentralization) and Algorithm 3 (decentralized ADMM
// beamforming, S x S branch).  On one GPU the antenna clusters are a batch
// axis: each (subcarrier, cluster) problem is a lane group of a wave64, the
// clusters of one subcarrier sit in one workgroup, and the consensus sum of the
// paper's fusion node is an LDS reduction in fixed cluster order (so every
// result is independent of how the work is tiled).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "dbp_device.h"
#include "dbp_launch.h"

namespace dbp {

constexpr int kStageRows = 8;   // rows of H_c staged per pass through LDS
// c32 slots of one wave's stage buffer: the staged rows, plus room for the
// padded transposes (a 32 x 32 float tile with a row pitch of 33, or two
// 16 x 16 problems as planes of 32 x 17 floats), whose offsets are then
// compile-time constants
constexpr int kStageWave = kStageRows * 64 + 32;

// Loads in the Gram prologues never branch: a request outside the problem
// (padding cluster, subcarrier past the end, ragged row past S) reads a valid
// address of the same array instead (row min(s, S-1) of a base clamped to the
// array start) and is zeroed by a select.
__device__ __forceinline__ c32 ld_or_zero(const c32* p, bool ok) {
  const c32 v = *p;
  return ok ? v : c32{0.f, 0.f};
}

// Fourth word of a raw buffer descriptor on gfx9-family GPUs (32-bit data
// format, no swizzle, stride 0: the range check is on bytes).
constexpr int kBufferWord3 = 0x00020000;

// Prefetch depth of the matrix-core Gram prologues (row pairs for U = 32, row
// quadruples for U = 16): the loads of the next chunk are in flight while the
// current chunk's MFMAs run.  Build-time tuning knobs.
#ifndef DBP_PREFETCH_U32
#define DBP_PREFETCH_U32 2
#endif
#ifndef DBP_PREFETCH_U16
#define DBP_PREFETCH_U16 1
#endif

// LDS carve-up shared by the kernels (all offsets in c32 units):
//   stage[nw][kStageWave]       staged H rows (kStageRows x 64, one slot per lane)
//   ystage[nw][kStageRows][8]   staged y entries (one per problem of the wave)
//   line[nw][64]                per-wave broadcast line
//   cons[2][nw][64]             double-buffered consensus slots (one per lane)
//   aux[nw][64]                 per-problem scalars (precoder power scaling)
struct Smem {
  c32* stage;
  c32* ystage;
  c32* line;
  c32* cons;
  c32* aux;
};

__device__ __forceinline__ Smem carve(c32* base, int nw) {
  Smem s;
  s.stage = base;
  s.ystage = s.stage + nw * kStageWave;
  s.line = s.ystage + nw * kStageRows * 8;
  s.cons = s.line + nw * 64;
  s.aux = s.cons + 2 * nw * 64;
  return s;
}

size_t smem_bytes(int nw) { return sizeof(c32) * (size_t)nw * (kStageWave + kStageRows * 8 + 64 + 128 + 64); }

// One pass over the S rows of H_c (and of y_c for symbol n): accumulates the
// Gram row A[v] += conj(H[s][u]) H[s][v] when WITH_GRAM, and always
// hy = sum_s conj(H[s][u]) y[s] (row u of H_c^H y_c).  BUF (U = 64, the one-shot
// detection): H through buffer loads, whose range check zeroes the rows past S; with
// a branch per row, the address registers that three waves per SIMD spill were
// waited for before every load (against stored factors, two waves, the branches
// measured up to 8 % faster).
template <int G, bool WITH_GRAM, bool BUF = false>
__device__ __forceinline__ c32 cluster_pass(const c32* __restrict__ H, const c32* __restrict__ y, c32 (&A)[G],
                                            int k, int c, int n, int u, int g, int lane, int wave, bool active,
                                            int B, int S, int U, int n_sym, const Smem& sm) {
  constexpr int R = kStageRows;
  c32 hy = cz();
  c32* stage = sm.stage + wave * kStageWave;
  c32* yst = sm.ystage + wave * R * 8;
  const c32* Hk = H + (size_t)k * B * U + (size_t)c * S * U;
  const c32* yk = y + ((size_t)k * n_sym + n) * B + (size_t)c * S;
  for (int s0 = 0; s0 < S; s0 += R) {
    c32 h[R];
    if constexpr (BUF) {
      static_assert(G == 64, "one problem per wave");
      const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
          const_cast<c32*>(Hk + (size_t)s0 * G), 0, active ? min(R, S - s0) * (G * 8) : 0, kBufferWord3);
#pragma unroll
      for (int r = 0; r < R; ++r)
        h[r] = __builtin_bit_cast(c32, __builtin_amdgcn_raw_buffer_load_b64(rs, r * (G * 8) + u * 8, 0, 0));
    } else {
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int s = s0 + r;
        h[r] = (active && s < S) ? Hk[(size_t)s * U + u] : cz();
      }
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (WITH_GRAM) stage[r * 64 + lane] = h[r];
    if (u < R) {
      const int s = s0 + u;
      yst[u * 8 + g] = (active && s < S) ? yk[s] : cz();
    }
    wave_lds_sync();
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if (WITH_GRAM) {
#pragma unroll
        for (int v0 = 0; v0 < G; v0 += 8) {
          c32 row[8];
          lds_read_vec<8>(stage + r * 64 + g * G + v0, row);
#pragma unroll
          for (int v = 0; v < 8; ++v) cmacc(A[v0 + v], h[r], row[v]);
        }
      }
      cmacc(hy, h[r], yst[r * 8 + g]);
    }
    wave_lds_sync();
  }
  return hy;
}

// Entries of the packed FP16 channel: a pair of binary16 values (real part in
// the low half), widened to FP32 exactly.
typedef _Float16 h16x2 __attribute__((ext_vector_type(2)));

// One complex entry scaled by 2^-e and rounded to complex FP16 (real part in
// the low half), the packed channel's format.
__device__ __forceinline__ uint32_t pack_pair(c32 v, int e) {
  const h16x2 p = {(_Float16)ldexpf(v.re, -e), (_Float16)ldexpf(v.im, -e)};
  return __builtin_bit_cast(uint32_t, p);
}

// The packed channel's exponent of a tile whose largest component is m: its
// largest component lands in [2^14, 2^15).
__device__ __forceinline__ int pack_exponent(float m) {
  return (m > 0.f && m <= 3.4028235e38f) ? min(max(ilogbf(m) - 14, -126), 113) : 0;
}

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off, 64));
  return v;
}
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

__device__ __forceinline__ c32 widen_h16(uint32_t w) {
  const h16x2 v = __builtin_bit_cast(h16x2, w);
  return c32{(float)v.x, (float)v.y};
}

// Row u of H_c^H y_c for symbol n for the resident forms (no Gram to share
// the pass with): every lane reads its column entry of each row of H_c
// (complex64, or the packed FP16 channel widened to FP32, the products
// accumulated in FP32 and the tile's power-of-two scale applied once at the
// end, which is exact) and the row's y entry directly (one address per lane
// group), with no LDS staging, so the loads of several rows are in flight
// together.  The FP16 channel uses it; for complex64 H the LDS-staged pass
// measured the same.
template <int G, bool H16>
__device__ __forceinline__ c32 cluster_hy_direct(const UlArgs& a, int k, int c, int n, int u, bool active) {
  c32 hy = cz();
  if (!active) return hy;
  const c32* yk = a.y + ((size_t)k * a.n_sym + n) * a.B + (size_t)c * a.S;
  const size_t hb = (size_t)k * a.B * G + (size_t)c * a.S * G + u;
  constexpr int CH = G >= 64 ? 4 : 8;   // rows in flight per lane (register budget at U = 64)
  int s = 0;
  for (; s + CH <= a.S; s += CH) {
    c32 hv[CH], yv[CH];
#pragma unroll
    for (int r = 0; r < CH; ++r) {
      if constexpr (H16)
        hv[r] = widen_h16(a.H16[hb + (size_t)(s + r) * G]);
      else
        hv[r] = a.H[hb + (size_t)(s + r) * G];
      yv[r] = yk[s + r];
    }
#pragma unroll
    for (int r = 0; r < CH; ++r) cmacc(hy, hv[r], yv[r]);
  }
  for (; s < a.S; ++s) {
    const c32 h = H16 ? widen_h16(a.H16[hb + (size_t)s * G]) : a.H[hb + (size_t)s * G];
    cmacc(hy, h, yk[s]);
  }
  if constexpr (H16) hy = cscale(hy, a.hscale[(size_t)k * a.C + c]);
  return hy;
}

typedef float f32x16 __attribute__((ext_vector_type(16)));

// Gauss-Jordan inversion of the HPD matrix B = G + rho I in the 32x32
// accumulator layout (lane l: column l%32, rows 8(r/4) + 4(l/32) + r%4), for
// the two Gram matrices of a wave, with lazy row and column scales: the stored
// matrix S relates to the partially swept one by true_ij = S_ij tau_i sigma_j,
// where a row / column not yet swept has scale 1 and sweeping pivot k (value
// d = B[k][k] of the current Schur complement) sets tau_k = 1/d and
// sigma_k = -1/d.  With these scales the sweep leaves row k and column k of S
// unchanged except for the diagonal, which becomes -d, and every other entry
// takes the plain Hermitian rank-1 update
//   S_ij -= conj(S_ki) S_kj / d,
// so S stays Hermitian throughout (the signed symmetry of the swept matrix is
// absorbed by the opposite signs of tau and sigma) and the multipliers of the
// update come from row k alone.  At the end every index is swept and
// B^{-1}_ij = -S_ij / (d_i d_j).
//
// Row k lives in register 4(k/8) + k%4 of lane half (k/4)&1.  On the FP32
// matrix cores the complex rank-1 update is two v_mfma_f32_32x32x2f32 whose
// K = 2 slots are the two lane halves, so row k is first copied into the
// other half (lanes < 32 get (Re, Im), lanes >= 32 (Im, Re)).
typedef float f32x16 __attribute__((ext_vector_type(16)));

// Undo the lazy scales of one swept 32x32 accumulator: entry (i, j) becomes
// -S_ij * pv_i * pv_j * extra, pv the reciprocal pivots.  pvv holds pv of this
// lane's column; the row factors come through 32 floats of wave-private LDS.
__device__ __forceinline__ void gj_unscale_u32(f32x16& re, f32x16& im, float pvv, float extra, int lane, float* line) {
  const int h = lane >> 5, col = lane & 31;
  if (h == 0) line[col] = pvv;
  wave_lds_sync();
  float4 q[4];
#pragma unroll
  for (int g = 0; g < 4; ++g) q[g] = *reinterpret_cast<const float4*>(line + 8 * g + 4 * h);
  wave_lds_sync();
  const float cs = -pvv * extra;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const float4 v = q[r / 4];
    const float pr = (r % 4 == 0) ? v.x : (r % 4 == 1) ? v.y : (r % 4 == 2) ? v.z : v.w;
    const float sc = cs * pr;
    re[r] *= sc;
    im[r] *= sc;
  }
}

// ADD_RHO: add rho to the diagonal first (false: the caller's accumulators
// already hold G + rho I).
template <bool ADD_RHO = true>
__device__ __forceinline__ void gj_invert_mfma_u32(f32x16 (&re)[2], f32x16 (&im)[2], int lane, float rho, float* line) {
  const int h = lane >> 5, col = lane & 31;
  if constexpr (ADD_RHO) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const bool dg = (8 * (r / 4) + 4 * h + (r % 4) == col);
      re[0][r] += dg ? rho : 0.f;
      re[1][r] += dg ? rho : 0.f;
    }
  } else {
    (void)rho;
  }
  float pvv[2] = {0.f, 0.f};
#pragma unroll
  for (int k = 0; k < 32; ++k) {
    const int rr = 4 * (k / 8) + (k % 4);   // register holding row k
    const int hk = (k / 4) & 1;             // lane half holding row k
    const bool isk = (col == k);
    const bool dg = isk && h == hk;
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const float sr = re[p][rr], si = im[p][rr];
      // Row k at column col with entry k zeroed (row and column k are left
      // alone by the update): lanes < 32 get (first, second) = (Re, Im),
      // lanes >= 32 (Im, Re).  A lane reads the lane of its own column in
      // either half, so zeroing at the source zeroes column k everywhere.
      // The imaginary update takes the same A operand and (Im, -Re) as B, so
      // the real part enters that swap negated.
      const float srm = isk ? 0.f : sr, sim = isk ? 0.f : si, srn = isk ? 0.f : -sr;
      const auto fs = __builtin_amdgcn_permlane32_swap(__float_as_uint(srm), __float_as_uint(sim), false, false);
      const auto sf = __builtin_amdgcn_permlane32_swap(__float_as_uint(sim), __float_as_uint(srn), false, false);
      const float first = __uint_as_float(fs[hk]);
      const float second = __uint_as_float(sf[hk]);
      const float d = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(sr), k + 32 * hk));
      const float pv = __builtin_amdgcn_rcpf(d);
      // Re: -pv (Re_i Re_j + Im_i Im_j), Im: -pv (Re_i Im_j - Im_i Re_j)
      const float Are = -pv * first;
      const float Aim = Are;
      re[p][rr] = dg ? -sr : sr;
      re[p] = __builtin_amdgcn_mfma_f32_32x32x2f32(Are, first, re[p], 0, 0, 0);
      im[p] = __builtin_amdgcn_mfma_f32_32x32x2f32(Aim, second, im[p], 0, 0, 0);
      pvv[p] = isk ? pv : pvv[p];
      // select in place (otherwise the compiler keeps every pivot's pv live
      // until the end)
      asm volatile("" : "+v"(pvv[p]));
    }
  }
#pragma unroll
  for (int p = 0; p < 2; ++p) gj_unscale_u32(re[p], im[p], pvv[p], 1.f, lane, line);
}

// Exchange between the wave's two 32-lane halves: v_permlane32_swap(X, Y)
// leaves [X of lanes 0-31 | Y of lanes 0-31] in its first result and
// [X of lanes 32-63 | Y of lanes 32-63] in its second.  With X and Y the two
// halves' accumulators of tile columns 0 and 1 (or problems 0 and 1), the
// first result is every lane's half-0 entry and the second its half-1 entry.
struct f32pair {
  float lo, hi;
};
__device__ __forceinline__ f32pair swap_halves(float x, float y) {
  const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
  return f32pair{__uint_as_float(s[0]), __uint_as_float(s[1])};
}

// v(lane) + v(lane ^ D) for D = 16 (odd and even rows of 16 lanes swapped by
// v_permlane16_swap) or D = 32 (wave halves, v_permlane32_swap); any other D
// goes through a lane shuffle.
template <int D>
__device__ __forceinline__ float pair_sum(float v) {
  if constexpr (D == 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
  } else if constexpr (D == 32) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
  } else {
    return v + __shfl_xor(v, D, 64);
  }
}

// Gram matrices of the two problems of a wave (U = 32, P = 2) on the matrix
// cores with v_mfma_f32_32x32x2f32, K running over pairs of antenna rows:
//   Re G = sum_s Hr[s]^T Hr[s] + Hi[s]^T Hi[s],
//   Im G = sum_s Hr[s]^T Hi[s] - Hi[s]^T Hr[s].
// For the Gram of one problem lane l supplies H[s0 + l/32][l%32] (or its
// P = Hr + Hi) as both the A and the B operand.  Only P^T P and M = Hr^T Hi
// are accumulated (two MFMAs per row pair instead of four), and
// Re G = P^T P - M - M^T, Im G = M - M^T are formed at the end.  The 32x32 result leaves lane l holding column l%32 for
// rows 8(r/4) + 4(l/32) + r%4 (r = 0..15); by Hermitian symmetry that is row
// l%32 conjugated, for half h = l/32 of the columns.  With INVERT the
// accumulators are replaced by (G + rho I)^{-1} on the matrix cores first.
// One exchange between lanes l and l^32 then gives every lane the full row of
// its own problem (lane-row layout, problem = l/32).  Returns row u of
// H_c^H y_c for symbol 0.
// PACK (factor-only kernel): when a.H16 is set, H is also written as the
// packed FP16 channel (a.H16, a.hscale; the format of pack_h16, bit for bit):
// the tile maxima are taken during the Gram's pass and one more pass converts.
template <bool INVERT, bool PACK = false>
__device__ __forceinline__ c32 gram_mfma_u32(const UlArgs& a, c32 (&A)[32], int lane, int wave, float* line,
                                             float* stage) {
  const int h = lane >> 5, col = lane & 31;
  f32x16 re[2], im[2];
  c32 hyp[2];
  const c32* Hp[2];
  const c32* yp[2];
  bool act[2];
  // With INVERT the real part starts from rho I: the diagonal entry (col, col)
  // sits in register 4 (col / 8) + col % 4 of lane half (col / 4) % 2.
  const int dr = (INVERT && h == ((col >> 2) & 1)) ? 4 * (col >> 3) + (col & 3) : -1;
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    const int lp = wave * 2 + p;
    const int ls = lp / a.Cp, c = lp % a.Cp;
    const int k = a.blk * a.sc_per_block + ls;
    act[p] = (k < a.n_sc) && (c < a.C);
    Hp[p] = act[p] ? a.H + (size_t)k * a.B * 32 + (size_t)c * a.S * 32 : a.H;
    yp[p] = act[p] ? a.y + (size_t)k * a.n_sym * a.B + (size_t)c * a.S : a.y;
#pragma unroll
    for (int r = 0; r < 16; ++r) re[p][r] = (r == dr) ? a.rho : 0.f;
    im[p] = f32x16{};
    hyp[p] = cz();
  }
  // Software pipeline: the loads of the next CH row pairs are in flight while
  // the MFMAs of the current ones run.
  constexpr int CH = DBP_PREFETCH_U32;
  c32 hv[2][CH], yv[2][CH], hn[2][CH], yn[2][CH];
  // Buffer loads over each problem's S rows of H_c and S entries of y_c (no
  // bytes for an inactive problem): the hardware range check returns zero
  // past the end, which pads the last row pair and the inactive problems
  // without a select, and the per-problem bases stay in scalar registers.
  // The whole offset is in the vector operand (the scalar offset is outside
  // the range check).
  __amdgpu_buffer_rsrc_t hrs[2], yrs[2];
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    hrs[p] = __builtin_amdgcn_make_buffer_rsrc(const_cast<c32*>(Hp[p]), 0, act[p] ? a.S * 256 : 0, kBufferWord3);
    yrs[p] = __builtin_amdgcn_make_buffer_rsrc(const_cast<c32*>(yp[p]), 0, act[p] ? a.S * 8 : 0, kBufferWord3);
  }
  auto fetch = [&](int s0, c32 (&hd)[2][CH], c32 (&yd)[2][CH]) {
#pragma unroll
    for (int q = 0; q < CH; ++q) {
      const int s = s0 + 2 * q + h;   // row s, column col: byte 256 s + 8 col
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        hd[p][q] = __builtin_bit_cast(c32, __builtin_amdgcn_raw_buffer_load_b64(hrs[p], s * 256 + col * 8, 0, 0));
        yd[p][q] = __builtin_bit_cast(c32, __builtin_amdgcn_raw_buffer_load_b64(yrs[p], s * 8, 0, 0));
      }
    }
  };
  const bool pk = PACK && a.H16 != nullptr;   // uniform
  float mx[2] = {0.f, 0.f};
  auto accumulate = [&](const c32 (&hd)[2][CH], const c32 (&yd)[2][CH]) {
#pragma unroll
    for (int q = 0; q < CH; ++q) {
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        const c32 x = hd[p][q];
        if constexpr (PACK)
          if (pk) mx[p] = fmaxf(mx[p], fmaxf(fabsf(x.re), fabsf(x.im)));
        const float pr = x.re + x.im;
        re[p] = __builtin_amdgcn_mfma_f32_32x32x2f32(pr, pr, re[p], 0, 0, 0);       // P^T P, P = Hr + Hi
        im[p] = __builtin_amdgcn_mfma_f32_32x32x2f32(x.re, x.im, im[p], 0, 0, 0);   // M = Hr^T Hi
        cmacc(hyp[p], x, yd[p][q]);
      }
    }
  };
  // the two buffers in turn (no copies).  INVERT: the loop body always runs
  // both halves and the rows past the last full double step follow it (with
  // an exit between the halves the compiler copies the accumulators of the
  // factor-only kernel on every step; the CG kernel is compiled best with the
  // exit)
  fetch(0, hv, yv);
  if constexpr (INVERT) {
    int s0 = 0;
    for (; s0 + 4 * CH <= a.S; s0 += 4 * CH) {
      fetch(s0 + 2 * CH, hn, yn);
      accumulate(hv, yv);
      fetch(s0 + 4 * CH, hv, yv);   // zeros past S
      accumulate(hn, yn);
    }
    if (s0 < a.S) {
      if (s0 + 2 * CH < a.S) fetch(s0 + 2 * CH, hn, yn);
      accumulate(hv, yv);
      if (s0 + 2 * CH < a.S) accumulate(hn, yn);
    }
  } else {
    for (int s0 = 0; s0 < a.S; s0 += 4 * CH) {
      if (s0 + 2 * CH < a.S) fetch(s0 + 2 * CH, hn, yn);
      accumulate(hv, yv);
      if (s0 + 2 * CH >= a.S) break;
      if (s0 + 4 * CH < a.S) fetch(s0 + 4 * CH, hv, yv);
      accumulate(hn, yn);
    }
  }
  if constexpr (PACK) {
    if (pk) {
      // rows of this lane's parity, both problems, four rows in flight
      uint32_t* h16 = const_cast<uint32_t*>(a.H16);
      int e[2];
#pragma unroll
      for (int p = 0; p < 2; ++p) e[p] = pack_exponent(wave_max(mx[p]));
      for (int s0 = h; s0 < a.S; s0 += 8) {
        c32 v[2][4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int s = s0 + 2 * t;
#pragma unroll
          for (int p = 0; p < 2; ++p) v[p][t] = ld_or_zero(Hp[p] + (size_t)min(s, a.S - 1) * 32 + col, true);
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int s = s0 + 2 * t;
#pragma unroll
          for (int p = 0; p < 2; ++p)
            if (act[p] && s < a.S) h16[(Hp[p] - a.H) + (size_t)s * 32 + col] = pack_pair(v[p][t], e[p]);
        }
      }
      if (lane == 0) {
#pragma unroll
        for (int p = 0; p < 2; ++p) {
          const int lp = wave * 2 + p;
          const int k = a.blk * a.sc_per_block + lp / a.Cp, c = lp % a.Cp;
          if (act[p]) const_cast<float*>(a.hscale)[(size_t)k * a.C + c] = ldexpf(1.f, e[p]);
        }
      }
    }
  }
  // re holds rho I + P^T P and im holds M = Hr^T Hi; since P^T P = Hr^T Hr
  // + Hi^T Hi + M + M^T, Re G = P^T P - M - M^T and Im G = M - M^T (two MFMAs
  // per row pair instead of three).  M goes through the wave's stage buffer
  // with a row pitch of 33 floats (entry (i, j) at 33 i + j), conflict-free
  // both for the row-wise write and the transposed read, and with a per-lane
  // base plus a compile-time offset for every register.
#pragma unroll
  for (int p = 0; p < 2; ++p) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int i = 8 * (r / 4) + 4 * h + (r % 4);
      stage[33 * i + col] = im[p][r];
    }
    wave_lds_sync();
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int i = 8 * (r / 4) + 4 * h + (r % 4);
      const float mt = stage[33 * col + i];
      re[p][r] -= im[p][r] + mt;
      im[p][r] -= mt;
    }
    wave_lds_sync();
  }
  if constexpr (INVERT) gj_invert_mfma_u32<false>(re, im, lane, a.rho, line);
  // exchange halves: lanes < 32 keep problem 0, lanes >= 32 keep problem 1
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int m0 = 8 * (r / 4) + (r % 4);      // column of this slot in half 0
    const f32pair xr = swap_halves(re[0][r], re[1][r]);
    const f32pair xi = swap_halves(im[0][r], im[1][r]);
    A[m0] = c32{xr.lo, -xi.lo};
    A[m0 + 4] = c32{xr.hi, -xi.hi};
  }
  // rows of parity 0 (first result) plus rows of parity 1 (second result)
  const f32pair yr = swap_halves(hyp[0].re, hyp[1].re);
  const f32pair yi = swap_halves(hyp[0].im, hyp[1].im);
  return c32{yr.lo + yr.hi, yi.lo + yi.hi};
}

// ---------------------------------------------------------------------------
// Mixed precision preprocessing for U = 32: the Gram on FP16 / BF16 matrix
// cores with FP32 accumulation.  Each problem's H_c is scaled by a power of two
// 2^e chosen from its largest entry (so its half-precision image uses the top
// of the format; exact, undone on the FP32 Gram), then split as
// H = H_hi + H_lo with H_hi = half(H) and H_lo = half(H - H_hi).  The Gram is
// refined to near FP32 accuracy by accumulating the correction products:
//   G ~ H_hi^H H_hi + H_hi^H H_lo + H_lo^H H_hi
// (the dropped H_lo^H H_lo term is below FP32 rounding for FP16).  Every
// v_mfma_f32_32x32x16 covers 16 real rows: lane l supplies column l%32 of the
// 8 rows 8(l/32) .. 8(l/32)+7 of its 16-row chunk as both the A and the B
// operand; the result uses the same 32x32 accumulator layout as the FP32 path.
// ---------------------------------------------------------------------------
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

template <typename HT>
struct HalfMma;
template <>
struct HalfMma<_Float16> {
  typedef f16x8 V;
  static __device__ __forceinline__ f32x16 mma(V x, V y, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(x, y, c, 0, 0, 0);
  }
};
template <>
struct HalfMma<__bf16> {
  typedef bf16x8 V;
  static __device__ __forceinline__ f32x16 mma(V x, V y, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, y, c, 0, 0, 0);
  }
};


// Normalisation of the mixed-mode Gram before the FP16 inverse.  H_c is scaled
// by 2^ex so that its largest entry lies in [2^13, 2^14); the Gram of i.i.d.
// entries then has diagonal about S * 2^24, and a shift of 9 + ceil(log2 S)
// brings it to about 2^15.  The FP16 inverse works on the operands r 2^-7 and
// 2^7 r / d of a pivot row r (both about 2^8 for entries of the diagonal's
// size, far below the FP16 limit of 2^16), so that values the matrix cores
// would flush (below 2^-14) only occur for contributions 2^-21 or more below
// the entries they update.  The shift
// depends on S only, so scaling H by 2^k changes ex alone and the result stays
// bit-exact.
__device__ __forceinline__ int norm_shift(int S) { return 9 + (32 - __builtin_clz((unsigned)(S > 1 ? S - 1 : 1))); }

// With NORM the Gram leaves scaled by 2^-norm_shift(S) instead of being
// returned to the units of H (see gj_invert_split16_u32); ex receives each
// problem's scaling exponent either way.
template <typename HT, bool NORM>
__device__ __forceinline__ void gram_split_u32(const UlArgs& a, f32x16 (&re)[2], f32x16 (&im)[2], c32 (&hyp)[2],
                                               int lane, int wave, int (&ex)[2], float* stage, float (&trg)[2]) {
  typedef typename HalfMma<HT>::V V;
  const int h = lane >> 5, col = lane & 31;
  const c32* Hp[2];
  const c32* yp[2];
  bool act[2];
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    const int lp = wave * 2 + p;
    const int ls = lp / a.Cp, c = lp % a.Cp;
    const int k = a.blk * a.sc_per_block + ls;
    act[p] = (k < a.n_sc) && (c < a.C);
    Hp[p] = act[p] ? a.H + (size_t)k * a.B * 32 + (size_t)c * a.S * 32 : a.H;
    yp[p] = act[p] ? a.y + (size_t)k * a.n_sym * a.B + (size_t)c * a.S : a.y;
    re[p] = f32x16{};
    im[p] = f32x16{};
    hyp[p] = cz();
  }
  // buffer loads over each problem's S rows (as in gram_mfma_u32)
  __amdgpu_buffer_rsrc_t hrs[2], yrs[2];
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    hrs[p] = __builtin_amdgcn_make_buffer_rsrc(const_cast<c32*>(Hp[p]), 0, act[p] ? a.S * 256 : 0, kBufferWord3);
    yrs[p] = __builtin_amdgcn_make_buffer_rsrc(const_cast<c32*>(yp[p]), 0, act[p] ? a.S * 8 : 0, kBufferWord3);
  }
  // pass 1: largest |Re|, |Im| of each problem -> scale exponent (and
  // ||H_c||_F^2 = tr(G_c))
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    float m = 0.f, ss = 0.f;
    for (int s0 = 0; s0 < a.S; s0 += 16) {
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const int s = s0 + 8 * h + t;
        const c32 v = __builtin_bit_cast(c32, __builtin_amdgcn_raw_buffer_load_b64(hrs[p], s * 256 + col * 8, 0, 0));
        m = fmaxf(m, fmaxf(fabsf(v.re), fabsf(v.im)));
        ss = fmaf(v.re, v.re, fmaf(v.im, v.im, ss));
      }
    }
    trg[p] = wave_sum(ss);
    m = wave_max(m);
    int x = 0;
    if (m > 0.f) frexpf(m, &x);      // m < 2^x
    ex[p] = 14 - x;                  // scaled entries stay below 2^14
  }
  // pass 2: split and accumulate
  for (int s0 = 0; s0 < a.S; s0 += 16) {
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      c32 v[8];
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const int s = s0 + 8 * h + t;
        v[t] = __builtin_bit_cast(c32, __builtin_amdgcn_raw_buffer_load_b64(hrs[p], s * 256 + col * 8, 0, 0));
        const c32 yv = __builtin_bit_cast(c32, __builtin_amdgcn_raw_buffer_load_b64(yrs[p], s * 8, 0, 0));
        cmacc(hyp[p], v[t], yv);
      }
      V rh, rl, ih, il;
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const float xr = ldexpf(v[t].re, ex[p]), xi = ldexpf(v[t].im, ex[p]);
        const HT hr = (HT)xr, hi = (HT)xi;
        rh[t] = hr;
        rl[t] = (HT)(xr - (float)hr);
        ih[t] = hi;
        il[t] = (HT)(xi - (float)hi);
      }
      // Re G = Hr^T Hr + Hi^T Hi
      re[p] = HalfMma<HT>::mma(rh, rh, re[p]);
      re[p] = HalfMma<HT>::mma(rh, rl, re[p]);
      re[p] = HalfMma<HT>::mma(rl, rh, re[p]);
      re[p] = HalfMma<HT>::mma(ih, ih, re[p]);
      re[p] = HalfMma<HT>::mma(ih, il, re[p]);
      re[p] = HalfMma<HT>::mma(il, ih, re[p]);
      // M = Hr^T Hi (Im G = M - M^T, below)
      im[p] = HalfMma<HT>::mma(rh, ih, im[p]);
      im[p] = HalfMma<HT>::mma(rh, il, im[p]);
      im[p] = HalfMma<HT>::mma(rl, ih, im[p]);
    }
  }
  // antisymmetrise through the stage buffer, as in gram_mfma_u32
#pragma unroll
  for (int p = 0; p < 2; ++p) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int i = 8 * (r / 4) + 4 * h + (r % 4);
      stage[33 * i + col] = im[p][r];
    }
    wave_lds_sync();
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int i = 8 * (r / 4) + 4 * h + (r % 4);
      im[p][r] -= stage[33 * col + i];
    }
    wave_lds_sync();
  }
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    const int sh = NORM ? norm_shift(a.S) : 2 * ex[p];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      re[p][r] = ldexpf(re[p][r], -sh);
      im[p][r] = ldexpf(im[p][r], -sh);
    }
  }
}

// Accumulator layout -> lane-row layout (lanes < 32: problem 0, >= 32: problem 1)
__device__ __forceinline__ void acc_to_rows_u32(const f32x16 (&re)[2], const f32x16 (&im)[2], c32 (&A)[32], int h) {
  (void)h;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int m0 = 8 * (r / 4) + (r % 4);
    const f32pair xr = swap_halves(re[0][r], re[1][r]);
    const f32pair xi = swap_halves(im[0][r], im[1][r]);
    A[m0] = c32{xr.lo, -xi.lo};
    A[m0 + 4] = c32{xr.hi, -xi.hi};
  }
}

// rows of parity 0 plus rows of parity 1 of H_c^H y_c, for this lane's problem
__device__ __forceinline__ c32 combine_hy(const c32 (&hyp)[2], int h) {
  (void)h;
  const f32pair yr = swap_halves(hyp[0].re, hyp[1].re);
  const f32pair yi = swap_halves(hyp[0].im, hyp[1].im);
  return c32{yr.lo + yr.hi, yi.lo + yi.hi};
}

// Regularised inverse in FP64 on the VALU (lane-row layout, rotated
// Gauss-Jordan as in gj_invert), for the poorly conditioned case U/S > 0.8.
struct c64 {
  double re, im;
};

template <int G>
__device__ __forceinline__ void gj_invert64(c64 (&A)[G], int u, c64* line) {
  for (int k = 0; k < G; ++k) {
    const double sg = (u < k) ? -1.0 : 1.0;
    line[(u - k) & (G - 1)] = c64{sg * A[0].re, -sg * A[0].im};
    wave_lds_sync();
    const double p = 1.0 / line[0].re;
    const bool me = (u == k);
    const c64 m = me ? c64{-p, 0.0} : c64{A[0].re * p, A[0].im * p};
    const c64 pivot_new = me ? c64{p, 0.0} : c64{-m.re, -m.im};
#pragma unroll
    for (int j0 = 0; j0 < G; j0 += 4) {
      c64 rk[4];
      const double2* q = reinterpret_cast<const double2*>(line + j0);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const double2 t = q[i];
        rk[i] = c64{t.x, t.y};
      }
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) {
        const int j = j0 + jj;
        if (j == 0) continue;
        c64 base = me ? c64{0.0, 0.0} : A[j];
        base.re = fma(-m.re, rk[jj].re, base.re);
        base.re = fma(m.im, rk[jj].im, base.re);
        base.im = fma(-m.re, rk[jj].im, base.im);
        base.im = fma(-m.im, rk[jj].re, base.im);
        A[j - 1] = base;
      }
    }
    A[G - 1] = pivot_new;
    wave_lds_sync();
  }
}

// ---------------------------------------------------------------------------
// Regularised inverse on the FP16 matrix cores (mixed modes): the sweep of
// gj_invert_mfma_u32 (lazy row / column scales, Hermitian update
// S_ij -= conj(S_ki) S_kj / d), with the rank-1 update issued as one
// v_mfma_f32_32x32x16_f16 per real / imaginary part.  The update is a_i b_j
// with a = -conj(r) 2^7 / d and b = r 2^-7 (r = row k): the same FP32
// coefficient 1/d as the FP32 sweep and its final unscaling, and two operands
// of comparable size (the power of two is exact).  Each operand is split into
// an FP16 hi + lo pair (round to nearest, about 22 significant bits together)
// and the K-terms hi.hi, hi.lo, lo.hi of the two real products take six of
// the eight K-slots of the lane half that holds row k: every operand a lane
// supplies comes from its own registers, and the other half supplies zeros,
// so nothing crosses lane halves.  Accumulation is FP32; the dropped lo.lo
// terms are 2^-22 relative.  FP16 MFMA runs beside the VALU, unlike FP32
// MFMA.  The matrix arrives normalised (norm_shift): rho is the normalised
// regulariser and post the power of two that undoes it.
// ---------------------------------------------------------------------------
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

// (x, y) -> packed FP16 pairs hi = (x_hi, y_hi) and lo = (x - x_hi, y - y_hi)
__device__ __forceinline__ void split_f16(float x, float y, unsigned& hi, unsigned& lo) {
  const f16x2 hv = f16x2{(_Float16)x, (_Float16)y};
  const f16x2 lv = f16x2{(_Float16)(x - (float)hv[0]), (_Float16)(y - (float)hv[1])};
  hi = __builtin_bit_cast(unsigned, hv);
  lo = __builtin_bit_cast(unsigned, lv);
}

__device__ __forceinline__ f16x8 as_f16x8(u32x4 v) { return __builtin_bit_cast(f16x8, v); }

// S += a (x) b from the split pairs ah / al = (Re a, Im a), bh / bl = (Re b, Im b).
// K-slot pairs (dwords): real part (Re a, -Im a).(Re b, Im b), imaginary part
// (Re a, Im a).(Im b, Re b).
__device__ __forceinline__ void rank1_split16(f32x16& re, f32x16& im, unsigned ah, unsigned al, unsigned bh,
                                              unsigned bl) {
  const unsigned ahc = ah ^ 0x80000000u, alc = al ^ 0x80000000u;
  const unsigned bhs = __builtin_amdgcn_alignbit(bh, bh, 16), bls = __builtin_amdgcn_alignbit(bl, bl, 16);
  re = __builtin_amdgcn_mfma_f32_32x32x16_f16(as_f16x8(u32x4{ahc, ahc, alc, 0u}), as_f16x8(u32x4{bh, bl, bh, 0u}), re,
                                              0, 0, 0);
  im = __builtin_amdgcn_mfma_f32_32x32x16_f16(as_f16x8(u32x4{ah, ah, al, 0u}), as_f16x8(u32x4{bhs, bls, bhs, 0u}), im,
                                              0, 0, 0);
}

__device__ __forceinline__ void gj_invert_split16_u32(f32x16 (&re)[2], f32x16 (&im)[2], int lane, const float (&rho)[2],
                                                      const float (&post)[2], float* line) {
  const int h = lane >> 5, col = lane & 31;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const bool dg = (8 * (r / 4) + 4 * h + (r % 4) == col);
    re[0][r] += dg ? rho[0] : 0.f;
    re[1][r] += dg ? rho[1] : 0.f;
  }
  float pvv[2] = {0.f, 0.f};
#pragma unroll
  for (int k = 0; k < 32; ++k) {
    const int rr = 4 * (k / 8) + (k % 4);   // register holding row k
    const int hk = (k / 4) & 1;             // lane half holding row k
    const bool isk = (col == k);
    const bool here = (h == hk);
    // operand masks (row k's half, column k excluded) with the 2^7 / 2^-7 balance
    const float ma = (here && !isk) ? 128.f : 0.f;
    const float mb = (here && !isk) ? 0.0078125f : 0.f;
    const float dn = (here && isk) ? -1.f : 1.f;
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const float sr = re[p][rr], si = im[p][rr];
      const float d = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(sr), k + 32 * hk));
      const float pv = __builtin_amdgcn_rcpf(d);
      const float t = pv * ma;
      unsigned ah, al, bh, bl;
      split_f16(-sr * t, si * t, ah, al);
      split_f16(sr * mb, si * mb, bh, bl);
      re[p][rr] = sr * dn;
      rank1_split16(re[p], im[p], ah, al, bh, bl);
      pvv[p] = isk ? pv : pvv[p];
    }
  }
#pragma unroll
  for (int p = 0; p < 2; ++p) gj_unscale_u32(re[p], im[p], pvv[p], post[p], lane, line);
}

// Mixed-precision Gram + regularised inverse for U = 32; returns row u of
// H_c^H y_c and leaves row u of (G + rho I)^{-1} in A.  INV selects the
// inverse: 0 FP32 matrix cores, 1 FP64 VALU, 2 split FP16 matrix cores.
template <typename HT, int INV>
__device__ __forceinline__ c32 gram_inv_mixed_u32(const UlArgs& a, c32 (&A)[32], int lane, int wave, c64* line64,
                                                  float& trg) {
  const int h = lane >> 5;
  f32x16 re[2], im[2];
  c32 hyp[2];
  int ex[2];
  float tr[2];
  gram_split_u32<HT, INV == 2>(a, re, im, hyp, lane, wave, ex, reinterpret_cast<float*>(line64), tr);
  trg = h ? tr[1] : tr[0];
  if (INV == 0) {
    gj_invert_mfma_u32(re, im, lane, a.rho, reinterpret_cast<float*>(line64));
    acc_to_rows_u32(re, im, A, h);
  } else if (INV == 2) {
    float rho_n[2], post[2];
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const int e = 2 * ex[p] - norm_shift(a.S);
      rho_n[p] = ldexpf(a.rho, e);
      post[p] = ldexpf(1.f, e);
    }
    gj_invert_split16_u32(re, im, lane, rho_n, post, reinterpret_cast<float*>(line64));
    acc_to_rows_u32(re, im, A, h);
  } else {
    acc_to_rows_u32(re, im, A, h);
    const int u = lane & 31;
    c64 D[32];
#pragma unroll
    for (int v = 0; v < 32; ++v) D[v] = c64{(double)A[v].re + ((v == u) ? (double)a.rho : 0.0), (double)A[v].im};
    gj_invert64<32>(D, u, line64 + h * 32);
#pragma unroll
    for (int v = 0; v < 32; ++v) A[v] = c32{(float)D[v].re, (float)D[v].im};
  }
  return combine_hy(hyp, h);
}

// Sums over the four lane groups of v0 .. v3, handed to lane groups 0 .. 3:
// v_permlane16_swap of (0, 1) and (2, 3) adds rows in pairs, v_permlane32_swap
// then adds the halves.
__device__ __forceinline__ float scatter_sum(float v0, float v1, float v2, float v3) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v0), __float_as_uint(v1), false, false);
  const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(v2), __float_as_uint(v3), false, false);
  const float s01 = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  const float s23 = __uint_as_float(b[0]) + __uint_as_float(b[1]);
  const auto c = __builtin_amdgcn_permlane32_swap(__float_as_uint(s01), __float_as_uint(s23), false, false);
  return __uint_as_float(c[0]) + __uint_as_float(c[1]);
}

// Gram matrices of the four problems of a wave for U = 16 (P = 4) on the
// matrix cores with v_mfma_f32_16x16x4f32, K running over quadruples of
// antenna rows: lane l supplies H[s0 + l/16][l%16] (or P = Hr + Hi) as both
// operands.  Only P^T P and M = Hr^T Hi are accumulated (two MFMAs per row
// quadruple instead of four); Re G = P^T P - M - M^T and Im G = M - M^T are
// formed in the transpose.  The
// 16x16 result leaves lane l holding column l%16 for rows 4(l/16) + r
// (r = 0..3) of every problem; by Hermitian symmetry that is row l%16
// conjugated, columns 4(l/16) .. 4(l/16)+3.  An LDS transpose (two problems
// per pass through the wave's stage buffer) gives lane 16p + u the full row u
// of problem p.  Returns row u of H_c^H y_c for symbol 0.
typedef float f32x4 __attribute__((ext_vector_type(4)));

// Regularised inverses of the four problems of a U = 16 wave on the matrix
// cores: v_mfma_f32_16x16x1f32 runs four independent 16 x 16 x 1 products, one
// per problem (block p of the A and B operands is lane group p, block p of the
// result is registers 4p .. 4p+3).  On entry re[p] holds P^T P + rho I and
// im[p] holds M = Hr^T Hi of problem p in the accumulator layout (lane
// 16 q + col, register r: row 4 q + r, column col), so that B = H^H H + rho I
// has Re B = P^T P - M - M^T and Im B = M - M^T (M^T through LDS).
//
// The sweep is the Hermitian Gauss-Jordan elimination with lazy scales: for
// each pivot k, S_ij -= conj(w_i) w_j / S_kk for i, j != k, where w is row k;
// row and column k are left alone and the diagonal is not negated, so that
// B^{-1} = 2 D - D S D with D = diag(pv) the pivot reciprocals.  One pivot is
// four rank-1 matrix-core updates of all four problems (real and imaginary
// parts), against 60 vector FMAs per lane for the same work.  Row k of every
// problem sits in lane group k / 4, register 4 p + k % 4: it reaches problem
// p's lane group through the wave's stage buffer.  Entry k of w is zeroed in
// both operands, which leaves row and column k alone.
//
// On return lane 16 p + u holds row u of problem p's S in A (S is Hermitian:
// read as column u, conjugated) and its pivot reciprocal pv_u in *pvl.
__device__ __forceinline__ void gj_invert_mfma_u16(f32x4 (&re)[4], f32x4 (&im)[4], c32 (&A)[16], int lane,
                                                   c32* stage, float* pvl) {
  const int q = lane >> 4, col = lane & 15;
  float* pm = reinterpret_cast<float*>(stage);   // M of the four problems, row pitch 17
#pragma unroll
  for (int p = 0; p < 4; ++p)
#pragma unroll
    for (int r = 0; r < 4; ++r) pm[(16 * p + 4 * q + r) * 17 + col] = im[p][r];
  wave_lds_sync();
  f32x16 sr, si;
#pragma unroll
  for (int p = 0; p < 4; ++p)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float mt = pm[(16 * p + col) * 17 + 4 * q + r];
      sr[4 * p + r] = re[p][r] - im[p][r] - mt;
      si[4 * p + r] = im[p][r] - mt;
    }
  wave_lds_sync();
  // row k through two float planes [lane group][problem][column] (the real
  // and imaginary registers need not be paired for the stores)
  float* wre = reinterpret_cast<float*>(stage);
  float* wim = wre + 256;
  float pvm = 0.f;
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const int g = k >> 2, rr = k & 3;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      wre[(4 * q + p) * 16 + col] = sr[4 * p + rr];
      wim[(4 * q + p) * 16 + col] = si[4 * p + rr];
    }
    wave_lds_sync();
    const c32 w = c32{wre[(4 * g + q) * 16 + col], wim[(4 * g + q) * 16 + col]};   // row k of problem q
    const float d = wre[(4 * g + q) * 16 + k];                                     // its pivot
    wave_lds_sync();
    const float pv = __builtin_amdgcn_rcpf(d);
    const bool isk = (col == k);
    const float wr = isk ? 0.f : w.re, wi = isk ? 0.f : w.im, nwr = isk ? 0.f : -w.re;
    // Re: -pv (wr_i wr_j + wi_i wi_j), Im: -pv (wr_i wi_j - wi_i wr_j)
    const float ar = -pv * wr, ai = -pv * wi;
    sr = __builtin_amdgcn_mfma_f32_16x16x1f32(ar, wr, sr, 0, 0, 0);
    sr = __builtin_amdgcn_mfma_f32_16x16x1f32(ai, wi, sr, 0, 0, 0);
    si = __builtin_amdgcn_mfma_f32_16x16x1f32(ar, wi, si, 0, 0, 0);
    si = __builtin_amdgcn_mfma_f32_16x16x1f32(ai, nwr, si, 0, 0, 0);
    // lane 16 p + u keeps pivot u of problem p (selected in place: otherwise
    // the compiler keeps every pivot's pv live until the end)
    pvm = isk ? pv : pvm;
    asm volatile("" : "+v"(pvm));
  }
  *pvl = pvm;
  // to rows, two problems per pass (two float planes of row pitch 17)
  float* pre = reinterpret_cast<float*>(stage);
  float* pim = pre + 32 * 17;
#pragma unroll
  for (int half = 0; half < 2; ++half) {
#pragma unroll
    for (int pp = 0; pp < 2; ++pp)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = 4 * q + r;
        pre[(16 * pp + i) * 17 + col] = sr[4 * (2 * half + pp) + r];
        pim[(16 * pp + i) * 17 + col] = si[4 * (2 * half + pp) + r];
      }
    wave_lds_sync();
    if ((q >> 1) == half) {
      const int pp = q & 1;
#pragma unroll
      for (int v = 0; v < 16; ++v) A[v] = c32{pre[(16 * pp + v) * 17 + col], -pim[(16 * pp + v) * 17 + col]};
    }
    wave_lds_sync();
  }
}

// RHO: the real part starts from rho I (the diagonal entry (col, col) sits in
// register col - 4 q of lane group q = col / 4), so A leaves as G + rho I.
// INV (with RHO): A leaves as the lazily scaled inverse S of G + rho I
// (gj_invert_mfma_u16) and *pvl as the pivot reciprocal of this lane's row.
template <bool RHO = false, bool INV = false>
__device__ __forceinline__ c32 gram_mfma_u16(const UlArgs& a, c32 (&A)[16], int lane, int wave, c32* stage,
                                             float* pvl = nullptr) {
  const int q = lane >> 4, col = lane & 15;
  const int dr = RHO ? col - 4 * q : -1;
  f32x4 re[4], im[4];
  c32 hyp[4];
  const c32* Hp[4];
  const c32* yp[4];
  bool act[4];
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const int lp = wave * 4 + p;
    const int ls = lp / a.Cp, c = lp % a.Cp;
    const int k = a.blk * a.sc_per_block + ls;
    act[p] = (k < a.n_sc) && (c < a.C);
    Hp[p] = act[p] ? a.H + (size_t)k * a.B * 16 + (size_t)c * a.S * 16 : a.H;
    yp[p] = act[p] ? a.y + (size_t)k * a.n_sym * a.B + (size_t)c * a.S : a.y;
    #pragma unroll
    for (int r = 0; r < 4; ++r) re[p][r] = (r == dr) ? a.rho : 0.f;
    im[p] = f32x4{};
    hyp[p] = cz();
  }
  constexpr int CH = DBP_PREFETCH_U16;   // row quadruples per prefetch chunk
  c32 hv[4][CH], yv[4][CH], hn[4][CH], yn[4][CH];
  // Buffer loads over each problem's S rows (as in gram_mfma_u32).
  __amdgpu_buffer_rsrc_t hrs[4], yrs[4];
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    hrs[p] = __builtin_amdgcn_make_buffer_rsrc(const_cast<c32*>(Hp[p]), 0, act[p] ? a.S * 128 : 0, kBufferWord3);
    yrs[p] = __builtin_amdgcn_make_buffer_rsrc(const_cast<c32*>(yp[p]), 0, act[p] ? a.S * 8 : 0, kBufferWord3);
  }
  auto fetch = [&](int s0, c32 (&hd)[4][CH], c32 (&yd)[4][CH]) {
#pragma unroll
    for (int j = 0; j < CH; ++j) {
      const int s = s0 + 4 * j + q;   // row s, column col: byte 128 s + 8 col
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        hd[p][j] = __builtin_bit_cast(c32, __builtin_amdgcn_raw_buffer_load_b64(hrs[p], s * 128 + col * 8, 0, 0));
        yd[p][j] = __builtin_bit_cast(c32, __builtin_amdgcn_raw_buffer_load_b64(yrs[p], s * 8, 0, 0));
      }
    }
  };
  auto accumulate = [&](const c32 (&hd)[4][CH], const c32 (&yd)[4][CH]) {
#pragma unroll
    for (int j = 0; j < CH; ++j) {
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        const c32 x = hd[p][j];
        const float pr = x.re + x.im;
        re[p] = __builtin_amdgcn_mfma_f32_16x16x4f32(pr, pr, re[p], 0, 0, 0);       // P^T P, P = Hr + Hi
        im[p] = __builtin_amdgcn_mfma_f32_16x16x4f32(x.re, x.im, im[p], 0, 0, 0);   // M = Hr^T Hi
        cmacc(hyp[p], x, yd[p][j]);
      }
    }
  };
  // two buffers used in turn (no copies): the next chunk's loads are in
  // flight while the current one is accumulated
  fetch(0, hv, yv);
  for (int s0 = 0; s0 < a.S; s0 += 8 * CH) {
    if (s0 + 4 * CH < a.S) fetch(s0 + 4 * CH, hn, yn);
    accumulate(hv, yv);
    if (s0 + 4 * CH >= a.S) break;
    if (s0 + 8 * CH < a.S) fetch(s0 + 8 * CH, hv, yv);
    accumulate(hn, yn);
  }
  // Transpose through LDS, two problems per pass: the real and imaginary
  // accumulators go to two float planes, entry (i, j) of problem pp at
  // (16 pp + i) 17 + j (a row pitch of 17: the column read and the transposed
  // read are conflict-free, and every offset is a compile-time constant).
  // re holds P^T P and im holds M = Hr^T Hi, so
  // Re G[v][col] = (P^T P)[v][col] - M[v][col] - M[col][v] and
  // Im G[v][col] = M[v][col] - M[col][v].
  float* pre = reinterpret_cast<float*>(stage);
  float* pim = pre + 32 * 17;
  if constexpr (INV) {
    gj_invert_mfma_u16(re, im, A, lane, stage, pvl);
  } else {
#pragma unroll
    for (int half = 0; half < 2; ++half) {
#pragma unroll
      for (int pp = 0; pp < 2; ++pp)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int i = 4 * q + r;
          pre[(16 * pp + i) * 17 + col] = re[2 * half + pp][r];
          pim[(16 * pp + i) * 17 + col] = im[2 * half + pp][r];
        }
      wave_lds_sync();
      if ((q >> 1) == half) {
        const int pp = q & 1;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const float gr = pre[(16 * pp + v) * 17 + col], gi = pim[(16 * pp + v) * 17 + col];
          const float mt = pim[(16 * pp + col) * 17 + v];
          A[v] = c32{gr - gi - mt, mt - gi};
        }
      }
      wave_lds_sync();
    }
  }
  // H_c^H y_c: the sum over the four row classes, problem p's to lane group p
  return c32{scatter_sum(hyp[0].re, hyp[1].re, hyp[2].re, hyp[3].re),
             scatter_sum(hyp[0].im, hyp[1].im, hyp[2].im, hyp[3].im)};
}

// ---------------------------------------------------------------------------
// U = 32, one-shot ADMM: the regularised Gram B in 16 x 16 blocks
//   B = [P Q; Q^H R],  Pi = P^{-1},  W = Pi Q,  Si = (R - Q^H W)^{-1},  X = W Si,
// applied without forming the rest of the inverse:
//   t = q_2 - W^H q_1,   B^{-1} q = [Pi q_1 - X t; Si t],
// which takes the multiply-adds of one 32 x 32 product.  On this hardware FP32
// matrix instructions do not run beside the vector units, so their time adds
// to the vector time, and the full 32 x 32 sweep was two thirds of the
// kernel: 128 of its 192 v_mfma_f32_32x32x2f32 (72 cycles each).  The blocks
// take 128 v_mfma_f32_16x16x1f32 (both problems at once; the first 16 pivots
// sweep P, Q and R, the others R alone) and 32 v_mfma_f32_16x16x4f32 (33 cycles
// each) instead, and the Gram skips the block below the diagonal.
// W and R - Q^H W come out of the sweep of P's pivots, not from products with
// the explicit Pi: those would lose a factor of P's condition number (on
// antenna-correlated channels, coefficient 0.9, ten times the sweep's error).
// The product X^H = Si W^H is of the form A^H B, for which a lane's accumulator
// registers are its operands: lane 16 q + c holds A[4 q + r][c] and
// B[4 q + r][c], and step r of the product takes rows 4 q + r, q = 0 .. 3, as
// its four K slots.
// ---------------------------------------------------------------------------
struct Tile16 {
  f32x4 re, im;
};

// X^H Y
__device__ __forceinline__ Tile16 tile_mul(const Tile16& X, const Tile16& Y) {
  Tile16 C{};
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    C.re = __builtin_amdgcn_mfma_f32_16x16x4f32(X.re[r], Y.re[r], C.re, 0, 0, 0);
    C.im = __builtin_amdgcn_mfma_f32_16x16x4f32(X.re[r], Y.im[r], C.im, 0, 0, 0);
    C.re = __builtin_amdgcn_mfma_f32_16x16x4f32(X.im[r], Y.im[r], C.re, 0, 0, 0);
    C.im = __builtin_amdgcn_mfma_f32_16x16x4f32(-X.im[r], Y.re[r], C.im, 0, 0, 0);
  }
  return C;
}

__device__ __forceinline__ f32x16 pack_tiles(const Tile16 (&T)[2]) {
  f32x16 s;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    s[r] = T[0].re[r];
    s[4 + r] = T[0].im[r];
    s[8 + r] = T[1].re[r];
    s[12 + r] = T[1].im[r];
  }
  return s;
}

// Inverses of the Hermitian positive definite 16 x 16 matrices P[0], P[1] (one of
// each problem of the wave): the sweep of gj_invert_mfma_u16 with the four blocks
// of v_mfma_f32_16x16x1f32 holding (Re P[0], Im P[0], Re P[1], Im P[1]).  Row k
// reaches the lane groups through wave-private LDS (lds: 160 floats), or with
// LANES through lane swaps (ten vector instructions more per pivot, half the
// latency; lds: 32 floats).
// BORDER: the pivots also sweep the blocks of [P Q; Q^H R]: Q leaves as P^{-1} Q
// and R as R - Q^H P^{-1} Q.
template <bool LANES, bool BORDER>
__device__ __forceinline__ void tile_sweep_pair(Tile16 (&P)[2], Tile16 (*Q)[2], Tile16 (*R)[2], int lane, float* lds) {
  static_assert(!(LANES && BORDER), "the border's rows go through LDS");
  const int q = lane >> 4, col = lane & 15;
  const bool odd = q & 1;   // this lane group is an imaginary block
  f32x16 s = pack_tiles(P), sq{}, sr{};
  if constexpr (BORDER) {
    sq = pack_tiles(*Q);
    sr = pack_tiles(*R);
  }
  float* wq = lds + col;                               // write: [block][column], P then Q
  const float* rq = lds + 16 * (q & 2) + col;          // read: real block of this lane group's problem
  const float* dq = lds + 16 * (q & 2);
  constexpr int kPv = LANES ? 0 : 128;
  float* pvs = lds + kPv + 8 * (q & 2);                // this problem's pivot reciprocals
  static_for<16>([&](auto kc) {
    constexpr int k = decltype(kc)::value, g = k >> 2, rr = k & 3;
    float w_re, w_im, q_re = 0.f, q_im = 0.f, d;
    if constexpr (LANES) {
      // problem 0's row on the lower and problem 1's on the upper wave half,
      // then from the even or odd row of 16 lanes to both
      auto spread = [&](float x, float y) {
        const f32pair h = swap_halves(x, y);
        const unsigned v = __float_as_uint(g < 2 ? h.lo : h.hi);
        return __uint_as_float(__builtin_amdgcn_permlane16_swap(v, v, false, false)[g & 1]);
      };
      w_re = spread(s[rr], s[8 + rr]);
      w_im = spread(s[4 + rr], s[12 + rr]);
      d = bcast16<k>(w_re);
    } else {
      if (q == g) {   // the lane group that holds row k
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          wq[16 * b] = s[4 * b + rr];
          if constexpr (BORDER) wq[64 + 16 * b] = sq[4 * b + rr];
        }
      }
      wave_lds_sync();
      w_re = rq[0];
      w_im = rq[16];
      d = dq[k];
      if constexpr (BORDER) {
        q_re = rq[64];
        q_im = rq[80];
      }
      wave_lds_sync();
    }
    const float pv = __builtin_amdgcn_rcpf(d);
    const bool isk = (col == k);
    const float wr = isk ? 0.f : w_re, wi = isk ? 0.f : w_im;
    const float ar = -pv * wr, ai = -pv * wi;
    // Re: -pv (wr_i wr_j + wi_i wi_j), Im: -pv (wr_i wi_j - wi_i wr_j)
    s = __builtin_amdgcn_mfma_f32_16x16x1f32(ar, odd ? wi : wr, s, 0, 0, 0);
    if constexpr (BORDER) {
      const float q1 = odd ? q_im : q_re, q2 = odd ? -q_re : q_im;
      sq = __builtin_amdgcn_mfma_f32_16x16x1f32(ar, q1, sq, 0, 0, 0);
      sr = __builtin_amdgcn_mfma_f32_16x16x1f32(-pv * q_re, q1, sr, 0, 0, 0);
      s = __builtin_amdgcn_mfma_f32_16x16x1f32(ai, odd ? -wr : wi, s, 0, 0, 0);
      sq = __builtin_amdgcn_mfma_f32_16x16x1f32(ai, q2, sq, 0, 0, 0);
      sr = __builtin_amdgcn_mfma_f32_16x16x1f32(-pv * q_im, q2, sr, 0, 0, 0);
    } else {
      s = __builtin_amdgcn_mfma_f32_16x16x1f32(ai, odd ? -wr : wi, s, 0, 0, 0);
    }
    if (col == 0) pvs[k] = pv;   // (no vector instruction per pivot)
  });
  // P^{-1} = 2 D - D S D and P^{-1} Q = D S_Q, D = diag(pv)
  wave_lds_sync();
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    const float pc = lds[kPv + 16 * p + col];
    const float4 v = *reinterpret_cast<const float4*>(lds + kPv + 16 * p + 4 * q);
    const float pr[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      // (one reciprocal after the other: their product leaves FP32 where the
      // Gram is below 1e-19 or above 1e19)
      const float dg = (4 * q + r == col) ? 2.f * pc : 0.f;
      P[p].re[r] = fmaf(pr[r], -pc * s[8 * p + r], dg);
      P[p].im[r] = pr[r] * (-pc * s[8 * p + 4 + r]);
      if constexpr (BORDER) {
        (*Q)[p].re[r] = pr[r] * sq[8 * p + r];
        (*Q)[p].im[r] = pr[r] * sq[8 * p + 4 + r];
        (*R)[p].re[r] = sr[8 * p + r];
        (*R)[p].im[r] = sr[8 * p + 4 + r];
      }
    }
  }
  wave_lds_sync();
}

// Registers v[m] of lane groups q -> registers v[q] of lane groups m (a 4 x 4
// transpose of register index and lane group).
__device__ __forceinline__ void transpose_groups(float (&v)[4]) {
  const f32pair a = swap_halves(v[0], v[2]), b = swap_halves(v[1], v[3]);
  const auto lo = __builtin_amdgcn_permlane16_swap(__float_as_uint(a.lo), __float_as_uint(b.lo), false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap(__float_as_uint(a.hi), __float_as_uint(b.hi), false, false);
  v[0] = __uint_as_float(lo[0]);
  v[1] = __uint_as_float(lo[1]);
  v[2] = __uint_as_float(hi[0]);
  v[3] = __uint_as_float(hi[1]);
}

// Gram and block factors of the two problems of a wave.  Lane 32 p + 16 h + u
// receives in A[0 .. 15] column u of Pi (h = 0) or W (h = 1) of problem p and in
// A[16 .. 31] column u of X^H (h = 0) or Si (h = 1): conjugated, the rows that
// block_matvec_u32 needs.  Returns entry 16 h + u of H_c^H y_c for symbol 0.
__device__ __forceinline__ c32 gram_blocks_u32(const UlArgs& a, c32 (&A)[32], int lane, int wave, float* stage) {
  const int q = lane >> 4, col = lane & 15;
  // P^T P (P = Hr + Hi) of the blocks (0, 0), (0, 1), (1, 1) and M = Hr^T Hi of
  // all four; the real diagonal starts from rho
  f32x4 pp[2][3], mm[2][4];
  c32 hyp[2][2];
  const c32* Hp[2];
  const c32* yp[2];
  bool act[2];
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    const int lp = wave * 2 + p;
    const int ls = lp / a.Cp, c = lp % a.Cp;
    const int k = a.blk * a.sc_per_block + ls;
    act[p] = (k < a.n_sc) && (c < a.C);
    Hp[p] = act[p] ? a.H + (size_t)k * a.B * 32 + (size_t)c * a.S * 32 : a.H;
    yp[p] = act[p] ? a.y + (size_t)k * a.n_sym * a.B + (size_t)c * a.S : a.y;
#pragma unroll
    for (int r = 0; r < 4; ++r) pp[p][0][r] = pp[p][2][r] = (4 * q + r == col) ? a.rho : 0.f;
    pp[p][1] = f32x4{};
#pragma unroll
    for (int t = 0; t < 4; ++t) mm[p][t] = f32x4{};
    hyp[p][0] = hyp[p][1] = cz();
  }
  // buffer loads over each problem's S rows (as in gram_mfma_u32): row s,
  // columns col and 16 + col at bytes 256 s + 8 col (+ 128)
  __amdgpu_buffer_rsrc_t hrs[2], yrs[2];
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    hrs[p] = __builtin_amdgcn_make_buffer_rsrc(const_cast<c32*>(Hp[p]), 0, act[p] ? a.S * 256 : 0, kBufferWord3);
    yrs[p] = __builtin_amdgcn_make_buffer_rsrc(const_cast<c32*>(yp[p]), 0, act[p] ? a.S * 8 : 0, kBufferWord3);
  }
  struct Rows {
    c32 h[2][2], y[2];   // [problem][column block], four rows (one per lane group)
  };
  auto fetch = [&](int s0, Rows& d) {
    const int s = s0 + q;
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      d.h[p][0] = __builtin_bit_cast(c32, __builtin_amdgcn_raw_buffer_load_b64(hrs[p], s * 256 + col * 8, 0, 0));
      d.h[p][1] = __builtin_bit_cast(c32, __builtin_amdgcn_raw_buffer_load_b64(hrs[p], s * 256 + 128 + col * 8, 0, 0));
      d.y[p] = __builtin_bit_cast(c32, __builtin_amdgcn_raw_buffer_load_b64(yrs[p], s * 8, 0, 0));
    }
  };
  auto accumulate = [&](const Rows& d) {
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const c32 x0 = d.h[p][0], x1 = d.h[p][1];
      const float s0 = x0.re + x0.im, s1 = x1.re + x1.im;
      pp[p][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(s0, s0, pp[p][0], 0, 0, 0);
      pp[p][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(s0, s1, pp[p][1], 0, 0, 0);
      pp[p][2] = __builtin_amdgcn_mfma_f32_16x16x4f32(s1, s1, pp[p][2], 0, 0, 0);
      mm[p][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(x0.re, x0.im, mm[p][0], 0, 0, 0);
      mm[p][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(x0.re, x1.im, mm[p][1], 0, 0, 0);
      mm[p][2] = __builtin_amdgcn_mfma_f32_16x16x4f32(x1.re, x0.im, mm[p][2], 0, 0, 0);
      mm[p][3] = __builtin_amdgcn_mfma_f32_16x16x4f32(x1.re, x1.im, mm[p][3], 0, 0, 0);
      cmacc(hyp[p][0], x0, d.y[p]);
      cmacc(hyp[p][1], x1, d.y[p]);
    }
  };
  // two buffers in turn: the loads of the next eight rows are in flight
  Rows d0, d1;
  fetch(0, d0);
  fetch(4, d1);
  int s0 = 0;
  for (; s0 + 4 < a.S; s0 += 8) {
    accumulate(d0);
    fetch(s0 + 8, d0);    // zeros past S
    accumulate(d1);
    fetch(s0 + 12, d1);
  }
  if (s0 < a.S) accumulate(d0);
  // Re G_IJ = (P^T P)_IJ - M_IJ - (M_JI)^T, Im G_IJ = M_IJ - (M_JI)^T: the
  // transposes of M_00, M_10 and M_11 through the stage buffer (row pitch 17)
  Tile16 P[2], Q[2], R[2];
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    constexpr int src[3] = {0, 2, 3};
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) stage[(16 * t + 4 * q + r) * 17 + col] = mm[p][src[t]][r];
    wave_lds_sync();
    f32x4 mt[3];
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) mt[t][r] = stage[(16 * t + col) * 17 + 4 * q + r];
    wave_lds_sync();
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      P[p].re[r] = pp[p][0][r] - (mm[p][0][r] + mt[0][r]);
      P[p].im[r] = mm[p][0][r] - mt[0][r];
      Q[p].re[r] = pp[p][1][r] - (mm[p][1][r] + mt[1][r]);
      Q[p].im[r] = mm[p][1][r] - mt[1][r];
      R[p].re[r] = pp[p][2][r] - (mm[p][3][r] + mt[2][r]);
      R[p].im[r] = mm[p][3][r] - mt[2][r];
    }
  }
  tile_sweep_pair<false, true>(P, &Q, &R, lane, stage);   // Pi, W and R - Q^H W
  Tile16 (&W)[2] = Q, V[2];
  // V = W^H, for X^H = Si W^H
#pragma unroll
  for (int p = 0; p < 2; ++p) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      stage[(4 * q + r) * 17 + col] = W[p].re[r];
      stage[(16 + 4 * q + r) * 17 + col] = W[p].im[r];
    }
    wave_lds_sync();
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      V[p].re[r] = stage[col * 17 + 4 * q + r];
      V[p].im[r] = -stage[(16 + col) * 17 + 4 * q + r];
    }
    wave_lds_sync();
  }
  tile_sweep_pair<false, false>(R, nullptr, nullptr, lane, stage);   // Si
  Tile16 X[2];
#pragma unroll
  for (int p = 0; p < 2; ++p) X[p] = tile_mul(R[p], V[p]);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    float l_re[4] = {P[0].re[r], W[0].re[r], P[1].re[r], W[1].re[r]};
    float l_im[4] = {P[0].im[r], W[0].im[r], P[1].im[r], W[1].im[r]};
    float h_re[4] = {X[0].re[r], R[0].re[r], X[1].re[r], R[1].re[r]};
    float h_im[4] = {X[0].im[r], R[0].im[r], X[1].im[r], R[1].im[r]};
    transpose_groups(l_re);
    transpose_groups(l_im);
    transpose_groups(h_re);
    transpose_groups(h_im);
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      A[4 * g + r] = c32{l_re[g], l_im[g]};
      A[16 + 4 * g + r] = c32{h_re[g], h_im[g]};
    }
  }
  return c32{scatter_sum(hyp[0][0].re, hyp[0][1].re, hyp[1][0].re, hyp[1][1].re),
             scatter_sum(hyp[0][0].im, hyp[0][1].im, hyp[1][0].im, hyp[1][1].im)};
}

// B^{-1} q from the blocks of gram_blocks_u32 (G = 32) or invert_blocks_u64 (G = 64):
// lane u of the problem's upper half (rows) holds column u of Pi and X^H, of the
// lower half of W and Si.  q_1 (and then t) reaches all lanes through the
// problem's part of the broadcast line.
template <int G>
__device__ __forceinline__ c32 block_matvec(const c32 (&A)[G], c32 q, c32* line, int gbase, int lane, bool upper) {
  constexpr int H = G / 2;
  // sum_v conj(A[v0 + v]) x_v, 16 entries at a time in the order of matvec16c
  auto mul = [&](int v0, const c32* x) -> c32 {
    c32 acc = cz();
#pragma unroll
    for (int j = 0; j < H; j += 16) {
      c32 s0 = cz(), s1 = cz();
#pragma unroll
      for (int i = 0; i < 16; i += 8) {
        c32 r[8];
        lds_read_vec<8>(x + j + i, r);
#pragma unroll
        for (int v = 0; v < 8; v += 2) {
          cmacc(s0, A[v0 + j + i + v], r[v]);
          cmacc(s1, A[v0 + j + i + v + 1], r[v + 1]);
        }
      }
      acc = j ? cadd(acc, cadd(s0, s1)) : cadd(s0, s1);
    }
    return acc;
  };
  line[lane] = q;
  wave_lds_sync();
  const c32 a = mul(0, line + gbase);         // Pi q_1 | W^H q_1
  const c32 t = csub(q, a);                   // (lower rows) q_2 - W^H q_1
  __builtin_amdgcn_wave_barrier();            // (a wave's accesses are in order)
  line[lane] = t;
  wave_lds_sync();
  const c32 b = mul(H, line + gbase + H);     // X t | Si t
  wave_lds_sync();
  return upper ? csub(a, b) : b;
}

// The same at U = 32 by row broadcasts: v_permlane16_swap hands q_1 (and then t) to
// both rows of 16 lanes, no LDS, the same bits.  A product's latency is shorter, but
// its multiply-adds take about a third longer than those on LDS operands, so it is
// taken while a SIMD has one wave or the products are few (line_products).  T = 40,
// four symbols, S = 32 (us, LDS | row broadcasts): C = 2, 600 subcarriers
// 126 | 111; C = 5, 4800 subcarriers 840 | 1055; T = 5, one symbol, C = 8, 4800:
// 145 | 141.  (At U = 64 the row broadcasts were slower throughout: T = 40, C = 8,
// 600 subcarriers, one symbol 329 us against 292.)
__device__ __forceinline__ c32 block_matvec_u32(const c32 (&A)[32], c32 q, bool upper) {
  auto dup = [](float v, int row) {
    const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(s[row]);
  };
  const c32 a = matvec16c<0>(A, c32{dup(q.re, 0), dup(q.im, 0)});     // Pi q_1 | W^H q_1
  const c32 t = csub(q, a);                                           // (lower rows) q_2 - W^H q_1
  const c32 b = matvec16c<16>(A, c32{dup(t.re, 1), dup(t.im, 1)});    // X t | Si t
  return upper ? csub(a, b) : b;
}

// Downlink S x S Gram A_c[a][b] = sum_u conj(Hu[a][u]) Hu[b][u] (S <= 16,
// U = 32 users as the contraction index, two problems per wave) on the matrix
// cores with v_mfma_f32_16x16x4f32: lane l supplies Hu[l%16][u0 + l/16] (or
// its P = Hr + Hi) as both operands; only P P^T and M = Hr Hi^T are
// accumulated (two MFMAs per four users instead of four).  The operands come
// from the register copy hcol (lane u of group g: Hu[i][u]) through LDS, so H
// is read from memory once.  Leaves T in the accumulator layout (lane l: column
// l % 16, rows 4 (l / 16) + r); M^T comes through the wave's stage buffer.
__device__ __forceinline__ void gram_dl_mfma_s16_u32(const c32 (&hcol)[16], Tile16 (&T)[2], int lane, int g, int u,
                                                     c32* stage) {
  const int q = lane >> 4, r16 = lane & 15;
  f32x4 re[2], im[2];
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    // problem p's tile (from the register copy hcol, zero past S) through
    // the stage buffer: entry (i, w) at 33 i + w (a row pitch of 33 complex
    // values: conflict-free, and every offset a compile-time constant)
    if (g == p) {
#pragma unroll
      for (int i = 0; i < 16; ++i) stage[i * 33 + u] = hcol[i];
    }
    wave_lds_sync();
    c32 x[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) x[j] = stage[r16 * 33 + q + 4 * j];
    wave_lds_sync();
    re[p] = f32x4{};
    im[p] = f32x4{};
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const float pr = x[j].re + x[j].im;
      re[p] = __builtin_amdgcn_mfma_f32_16x16x4f32(pr, pr, re[p], 0, 0, 0);               // P P^T, P = Hr + Hi
      im[p] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[j].re, x[j].im, im[p], 0, 0, 0);   // M = Hr Hi^T
    }
  }
  // Re G[i][j] = (P P^T)[i][j] - M[i][j] - M[j][i], Im G[i][j] = M[i][j] - M[j][i]
  float* st = reinterpret_cast<float*>(stage);
#pragma unroll
  for (int p = 0; p < 2; ++p)
#pragma unroll
    for (int r = 0; r < 4; ++r) st[(16 * p + 4 * q + r) * 17 + r16] = im[p][r];
  wave_lds_sync();
#pragma unroll
  for (int p = 0; p < 2; ++p)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float mt = st[(16 * p + r16) * 17 + 4 * q + r];
      T[p].re[r] = re[p][r] - im[p][r] - mt;
      T[p].im[r] = im[p][r] - mt;
    }
  wave_lds_sync();
}

// Two problems' Hermitian tiles -> the split-row layout of matvec_split16: lane r
// of row h of 16 lanes of the problem's group gets entries 8 h .. 8 h + 7 of row r
// (column r conjugated; lane groups 2 h and 2 h + 1 hold its quarters).
__device__ __forceinline__ void tiles_to_split_rows(const Tile16 (&T)[2], c32 (&A)[8]) {
  auto pick = [](float x, float y, float& o0, float& o1) {
    const f32pair ab = swap_halves(x, y);
    const auto o = __builtin_amdgcn_permlane16_swap(__float_as_uint(ab.lo), __float_as_uint(ab.hi), false, false);
    o0 = __uint_as_float(o[0]);
    o1 = __uint_as_float(o[1]);
  };
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    pick(T[0].re[r], T[1].re[r], A[r].re, A[4 + r].re);
    pick(-T[0].im[r], -T[1].im[r], A[r].im, A[4 + r].im);
  }
}

// The inverses of gram_dl_mfma_s16_u32 shifted by tau (identity past S), in
// split rows.  MFMA: the sweep on the matrix cores (tile_sweep_pair), shorter
// where two waves share a SIMD (the budgeted form, 240 -> 214 us at B=256 U=32
// C=16, 1200 subcarriers); with four waves per SIMD the vector sweep on the split
// rows measured faster (1.31 against 1.36-1.38 ms per 38,400 subcarriers).
template <bool MFMA>
__device__ __forceinline__ void shift_invert_s16(Tile16 (&T)[2], float tau0, float tau1, int S, c32 (&A)[8], int lane,
                                                 c32* line) {
  const int q = lane >> 4, col = lane & 15;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const bool dg = 4 * q + r == col;
    T[0].re[r] += dg ? (col < S ? tau0 : 1.f) : 0.f;
    T[1].re[r] += dg ? (col < S ? tau1 : 1.f) : 0.f;
  }
  if constexpr (MFMA) tile_sweep_pair<true, false>(T, nullptr, nullptr, lane, reinterpret_cast<float*>(line));
  tiles_to_split_rows(T, A);
  if constexpr (!MFMA) gj_invert_sym_split16(A, col, q & 1, line + (lane & 32));
}

// ---------------------------------------------------------------------------
// U = 64 (one problem per wave): the 64x64 Gram and its regularised inverse as
// four 32x32 accumulator tiles (I, J) (rows 32I.., columns 32J..; lane l holds
// column 32J + l%32 of tile (I, J) for rows 32I + 8(r/4) + 4(l/32) + r%4).
// Gram: lane l supplies H[s0 + l/32][32I + l%32] as A and H[s0 + l/32][32J + l%32]
// as B.  Gauss-Jordan as in gj_invert_mfma_u32, with the rank-1 update of every
// pivot issued on all four tiles.
// ---------------------------------------------------------------------------
// Undo the lazy scales of the four swept tiles (as gj_unscale_u32): pvv[J]
// holds pv of column 32J + l%32; the 64 row factors go through LDS.
__device__ __forceinline__ void gj_unscale_u64(f32x16 (&re)[2][2], f32x16 (&im)[2][2], const float (&pvv)[2],
                                               float extra, int lane, float* line) {
  const int h = lane >> 5, col = lane & 31;
  line[32 * h + col] = pvv[h];
  wave_lds_sync();
  const float cs[2] = {-pvv[0] * extra, -pvv[1] * extra};
#pragma unroll
  for (int I = 0; I < 2; ++I) {
    float4 q[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) q[g] = *reinterpret_cast<const float4*>(line + 32 * I + 8 * g + 4 * h);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float4 v = q[r / 4];
      const float pr = (r % 4 == 0) ? v.x : (r % 4 == 1) ? v.y : (r % 4 == 2) ? v.z : v.w;
#pragma unroll
      for (int J = 0; J < 2; ++J) {
        const float sc = cs[J] * pr;
        re[I][J][r] *= sc;
        im[I][J][r] *= sc;
      }
    }
  }
  wave_lds_sync();
}

// dst = src^H for one 32x32 tile pair (real, imaginary) through the wave's
// stage buffer, a row pitch of 33 floats (as the Gram's transposes).
__device__ __forceinline__ void tile_conj_transpose(const f32x16& sre, const f32x16& sim, f32x16& dre, f32x16& dim,
                                                    int h, int col, float* stage) {
#pragma unroll
  for (int part = 0; part < 2; ++part) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int i = 8 * (r / 4) + 4 * h + (r % 4);
      stage[33 * i + col] = part ? sim[r] : sre[r];
    }
    wave_lds_sync();
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int i = 8 * (r / 4) + 4 * h + (r % 4);
      const float t = stage[33 * col + i];
      if (part)
        dim[r] = -t;
      else
        dre[r] = t;
    }
    wave_lds_sync();
  }
}

// X^H Y for 32 x 32 accumulator tiles (real and imaginary parts): register r of
// both operands holds one row per lane half, the two K slots of a step.
__device__ __forceinline__ void acc_mul(const f32x16& xr, const f32x16& xi, const f32x16& yr, const f32x16& yi,
                                        f32x16& cr, f32x16& ci) {
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    cr = __builtin_amdgcn_mfma_f32_32x32x2f32(xr[r], yr[r], cr, 0, 0, 0);
    ci = __builtin_amdgcn_mfma_f32_32x32x2f32(xr[r], yi[r], ci, 0, 0, 0);
    cr = __builtin_amdgcn_mfma_f32_32x32x2f32(xi[r], yi[r], cr, 0, 0, 0);
    ci = __builtin_amdgcn_mfma_f32_32x32x2f32(-xi[r], yr[r], ci, 0, 0, 0);
  }
}

// U = 64: B = G + rho I as 32 x 32 blocks [P Q; Q^H R] (accumulator tiles (0, 0),
// (0, 1), (1, 1); (1, 0) is not read), factored as at U = 32 (gram_blocks_u32).
// The first 32 pivots sweep all three tiles (six 32x32x2 instructions each) and
// leave Pi, W and R - Q^H W, the other 32 sweep the last tile alone (two); the
// product X^H = Si W^H takes 64.  The sweep keeps lazy row and column scales
// (see gj_invert_mfma_u32) and does not negate the diagonal.  Against the sweep
// of the whole matrix (six per pivot throughout): 320 instead of 384, half the
// vector instructions in the second half, and on ill-conditioned clusters a
// smaller error.
// FULL: A receives row u of B^{-1} (one more product, Pi + X W^H).  Otherwise
// lane u < 32 receives column u of Pi in A[0 .. 31] and of X^H in A[32 .. 63],
// lane 32 + u column u of W and of Si, for block_matvec.  f2 (may be null):
// ||B^{-1}||_F^2.
template <bool FULL>
__device__ __forceinline__ void invert_blocks_u64(f32x16 (&re)[2][2], f32x16 (&im)[2][2], int lane, float rho,
                                                  float* line, float* stage, c32 (&A)[64], float* f2) {
  const int h = lane >> 5, col = lane & 31;
  // B = G + rho I
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const bool dg = (8 * (r / 4) + 4 * h + (r % 4) == col);
    re[0][0][r] += dg ? rho : 0.f;
    re[1][1][r] += dg ? rho : 0.f;
  }
#pragma unroll
  for (int kk = 0; kk < 64; ++kk) {
    const int Ik = kk / 32, kr = kk % 32;
    const int rr = 4 * (kr / 8) + (kr % 4);
    const int hk = (kr / 4) & 1;
    const float d = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(re[Ik][Ik][rr]), kr + 32 * hk));
    const float pv = __builtin_amdgcn_rcpf(d);
    const bool isk = (col == kr);
    float first[2], second[2], At[2];
#pragma unroll
    for (int J = 0; J < 2; ++J) {
      if (J < Ik) continue;
      // row kk on both lane halves, entry kk zeroed at the source lanes
      // (lanes < 32 get (Re, Im), lanes >= 32 (Im, Re), with (Im, -Re) as the
      // imaginary update's B operand)
      const bool z = isk && J == Ik;
      const float sr = re[Ik][J][rr], si = im[Ik][J][rr];
      const float srm = z ? 0.f : sr, sim = z ? 0.f : si, srn = z ? 0.f : -sr;
      const auto fs = __builtin_amdgcn_permlane32_swap(__float_as_uint(srm), __float_as_uint(sim), false, false);
      const auto sf = __builtin_amdgcn_permlane32_swap(__float_as_uint(sim), __float_as_uint(srn), false, false);
      first[J] = __uint_as_float(fs[hk]);
      second[J] = __uint_as_float(sf[hk]);
      At[J] = -pv * first[J];
    }
#pragma unroll
    for (int I = 0; I < 2; ++I)
#pragma unroll
      for (int J = I; J < 2; ++J) {
        if (I < Ik) continue;
        re[I][J] = __builtin_amdgcn_mfma_f32_32x32x2f32(At[I], first[J], re[I][J], 0, 0, 0);
        im[I][J] = __builtin_amdgcn_mfma_f32_32x32x2f32(At[I], second[J], im[I][J], 0, 0, 0);
      }
    if (lane == 0) line[kk] = pv;
  }
  wave_lds_sync();
  // Pi and Si: 2 D - D S D, W: D S (rows)
#pragma unroll
  for (int I = 0; I < 2; ++I) {
    const float pc = line[32 * I + col];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const float4 v = *reinterpret_cast<const float4*>(line + 32 * I + 8 * g + 4 * h);
      const float pr[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int r = 4 * g + t;
        // (one reciprocal after the other, as in tile_sweep_pair)
        const float dg = (8 * g + 4 * h + t == col) ? 2.f * pc : 0.f;
        re[I][I][r] = fmaf(pr[t], -pc * re[I][I][r], dg);
        im[I][I][r] = pr[t] * (-pc * im[I][I][r]);
        if (I == 0) {
          re[0][1][r] *= pr[t];
          im[0][1][r] *= pr[t];
        }
      }
    }
  }
  wave_lds_sync();
  // X^H = Si W^H into tile (1, 0)
  f32x16 vr, vi;
  tile_conj_transpose(re[0][1], im[0][1], vr, vi, h, col, stage);
  re[1][0] = im[1][0] = f32x16{};
  acc_mul(re[1][1], im[1][1], vr, vi, re[1][0], im[1][0]);
  if constexpr (FULL) {
    acc_mul(re[1][0], im[1][0], vr, vi, re[0][0], im[0][0]);   // Pi + X W^H
    tile_conj_transpose(re[1][0], im[1][0], re[0][1], im[0][1], h, col, stage);   // X
  } else if (f2) {
    f32x16 tr = re[0][0], ti = im[0][0];
    acc_mul(re[1][0], im[1][0], vr, vi, tr, ti);
    float n = 0.f, off = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      n = fmaf(tr[r], tr[r], fmaf(ti[r], ti[r], n));
      n = fmaf(re[1][1][r], re[1][1][r], fmaf(im[1][1][r], im[1][1][r], n));
      off = fmaf(re[1][0][r], re[1][0][r], fmaf(im[1][0][r], im[1][0][r], off));
    }
    *f2 = group_sum<64>(fmaf(2.f, off, n));
  }
  // to lanes: column u of the left tile to lane u, of the right one to lane 32 + u
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int m0 = 8 * (r / 4) + (r % 4);
    const f32pair lr = swap_halves(re[0][0][r], FULL ? -re[0][1][r] : re[0][1][r]);
    const f32pair hr = swap_halves(FULL ? -re[1][0][r] : re[1][0][r], re[1][1][r]);
    // FULL: rows (columns conjugated)
    const f32pair li = swap_halves(FULL ? -im[0][0][r] : im[0][0][r], im[0][1][r]);
    const f32pair hi = swap_halves(im[1][0][r], FULL ? -im[1][1][r] : im[1][1][r]);
    A[m0] = c32{lr.lo, li.lo};
    A[m0 + 4] = c32{lr.hi, li.hi};
    A[32 + m0] = c32{hr.lo, hi.lo};
    A[32 + m0 + 4] = c32{hr.hi, hi.hi};
  }
}

// accumulator tiles -> lane-row layout: lane u < 32 takes column u of tile
// column 0, lane 32 + u column u of tile column 1 (conjugated into rows)
__device__ __forceinline__ void acc_to_rows_u64(const f32x16 (&re)[2][2], const f32x16 (&im)[2][2], c32 (&A)[64],
                                                int h) {
#pragma unroll
  for (int I = 0; I < 2; ++I)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int m0 = 32 * I + 8 * (r / 4) + (r % 4);
      const f32pair xr = swap_halves(re[I][0][r], re[I][1][r]);
      const f32pair xi = swap_halves(im[I][0][r], im[I][1][r]);
      A[m0] = c32{xr.lo, -xi.lo};
      A[m0 + 4] = c32{xr.hi, -xi.hi};
    }
  (void)h;
}

// lane u < 32 owns entry u of H_c^H y_c, lane 32 + u entry 32 + u; e0 / e1 are
// this lane's partial sums of entries col / 32 + col over its half of the rows
__device__ __forceinline__ c32 combine_hy_u64(c32 e0, c32 e1, int h) {
  (void)h;
  const f32pair yr = swap_halves(e0.re, e1.re);
  const f32pair yi = swap_halves(e0.im, e1.im);
  return c32{yr.lo + yr.hi, yi.lo + yi.hi};
}

// A cluster's S x 64 uplink block of a downlink problem, entry (antenna a, user w),
// in either layout of H (zero past S).
struct DlBlock64 {
  __amdgpu_buffer_rsrc_t rs;
  int S, sa, su;   // strides in bytes
  __device__ __forceinline__ c32 at(int a, int w) const {
    return __builtin_bit_cast(c32, __builtin_amdgcn_raw_buffer_load_b64(rs, a < S ? a * sa + w * su : (int)0x80000000u, 0, 0));
  }
};

// INVERT: 0 the Gram (rows of G in A), 1 its block factors, 2 rows of the inverse.
template <int INVERT, bool DL = false>
__device__ __forceinline__ c32 gram_mfma_u64(const UlArgs& a, c32 (&A)[64], int lane, int wave, float* line,
                                             float* stage, const DlBlock64* dl = nullptr) {
  const int h = lane >> 5, col = lane & 31;
  f32x16 re[2][2], im[2][2];
  c32 hy0 = cz(), hy1 = cz();
  const int ls = wave / a.Cp, c = wave % a.Cp;
  const int k = a.blk * a.sc_per_block + ls;
  const bool act = (k < a.n_sc) && (c < a.C);
  const c32* Hk = act ? a.H + (size_t)k * a.B * 64 + (size_t)c * a.S * 64 : a.H;
  const c32* yk = act ? a.y + (size_t)k * a.n_sym * a.B + (size_t)c * a.S : a.y;
#pragma unroll
  for (int I = 0; I < 2; ++I)
#pragma unroll
    for (int J = 0; J < 2; ++J) {
      re[I][J] = f32x16{};
      im[I][J] = f32x16{};
    }
  // buffer loads over the problem's S rows (as in gram_mfma_u32)
  const __amdgpu_buffer_rsrc_t hrs = __builtin_amdgcn_make_buffer_rsrc(const_cast<c32*>(Hk), 0, act ? a.S * 512 : 0, kBufferWord3);
  const __amdgpu_buffer_rsrc_t yrs = __builtin_amdgcn_make_buffer_rsrc(const_cast<c32*>(yk), 0, act ? a.S * 8 : 0, kBufferWord3);
  struct Rows {
    c32 x0, x1, y;   // two rows, one per lane half
  };
  auto fetch = [&](int s0, Rows& d) {
    const int s = s0 + h;   // row s, columns col and 32 + col: bytes 512 s + 8 col (+ 256)
    if constexpr (DL) {
      d.x0 = dl->at(col, s);
      d.x1 = dl->at(32 + col, s);
      d.y = cz();
      return;
    }
    d.x0 = __builtin_bit_cast(c32, __builtin_amdgcn_raw_buffer_load_b64(hrs, s * 512 + col * 8, 0, 0));
    d.x1 = __builtin_bit_cast(c32, __builtin_amdgcn_raw_buffer_load_b64(hrs, s * 512 + 256 + col * 8, 0, 0));
    d.y = __builtin_bit_cast(c32, __builtin_amdgcn_raw_buffer_load_b64(yrs, s * 8, 0, 0));
  };
  auto accumulate = [&](const Rows& d) {
    const c32 xs[2] = {d.x0, d.x1};
    const float ps[2] = {d.x0.re + d.x0.im, d.x1.re + d.x1.im};
#pragma unroll
    for (int I = 0; I < 2; ++I)
#pragma unroll
      for (int J = 0; J < 2; ++J) {
        // with INVERT tile (1, 0) of G is not read: its P^T P part is not accumulated
        if (!(INVERT && I == 1 && J == 0))
          re[I][J] = __builtin_amdgcn_mfma_f32_32x32x2f32(ps[I], ps[J], re[I][J], 0, 0, 0);        // P^T P
        im[I][J] = __builtin_amdgcn_mfma_f32_32x32x2f32(xs[I].re, xs[J].im, im[I][J], 0, 0, 0);   // M
      }
    // entries col and 32 + col of H_c^H y_c over the rows of this lane's parity
    cmacc(hy0, d.x0, d.y);
    cmacc(hy1, d.x1, d.y);
  };
  // Four buffers in turn, eight rows in flight: with two waves per SIMD a step's
  // matrix instructions (about 900 cycles for both) are shorter than a load
  // from memory.
  Rows d[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) fetch(2 * j, d[j]);   // zeros past S
  int s0 = 0;
  for (; s0 + 8 <= a.S; s0 += 8) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      accumulate(d[j]);
      fetch(s0 + 8 + 2 * j, d[j]);
    }
  }
#pragma unroll
  for (int j = 0; j < 4; ++j)
    if (s0 + 2 * j < a.S) accumulate(d[j]);   // uniform
  // Tile (I, J) holds P^T P and M = Hr^T Hi restricted to rows 32 I.. and
  // columns 32 J..; Re G_IJ = (P^T P)_IJ - M_IJ - (M_JI)^T and
  // Im G_IJ = M_IJ - (M_JI)^T.  The transposes go through the wave's stage
  // buffer, one 32 x 32 tile at a time, with a row pitch of 33 as for U = 32;
  // both off-diagonal transposes are read before either off-diagonal tile
  // changes.
  auto transposed = [&](const f32x16& m, float (&out)[16]) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int i = 8 * (r / 4) + 4 * h + (r % 4);
      stage[33 * i + col] = m[r];
    }
    wave_lds_sync();
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int i = 8 * (r / 4) + 4 * h + (r % 4);
      out[r] = stage[33 * col + i];
    }
    wave_lds_sync();
  };
  {
    float t01[16] = {}, t10[16];
    if constexpr (INVERT == 0) transposed(im[0][1], t01);
    transposed(im[1][0], t10);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      re[0][1][r] -= im[0][1][r] + t10[r];
      im[0][1][r] -= t10[r];
      if (!INVERT) {
        re[1][0][r] -= im[1][0][r] + t01[r];
        im[1][0][r] -= t01[r];
      }
    }
  }
#pragma unroll
  for (int D = 0; D < 2; ++D) {
    float td[16];
    transposed(im[D][D], td);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      re[D][D][r] -= im[D][D][r] + td[r];
      im[D][D][r] -= td[r];
    }
  }
  if constexpr (INVERT != 0)
    invert_blocks_u64<INVERT == 2>(re, im, lane, a.rho, line, stage, A, nullptr);
  else
    acc_to_rows_u64(re, im, A, h);
  return combine_hy_u64(hy0, hy1, h);
}

// Split-FP16 Gauss-Jordan inverse for U = 64 (four 32x32 tiles, one problem
// per wave), as gj_invert_split16_u32: the pivot row kk lives in tile row Ik,
// half hk of tiles (Ik, 0) and (Ik, 1); with the Hermitian stored matrix the
// operand a of tile row I comes from tile (Ik, I) and b of tile column J from
// tile (Ik, J), all in half hk, so each of the four tile updates is two FP16
// MFMAs built from lane-local registers.
__device__ __forceinline__ void gj_invert_split16_u64(f32x16 (&re)[2][2], f32x16 (&im)[2][2], int lane, float rho,
                                                      float post, float* line) {
  const int h = lane >> 5, col = lane & 31;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const bool dg = (8 * (r / 4) + 4 * h + (r % 4) == col);
    re[0][0][r] += dg ? rho : 0.f;
    re[1][1][r] += dg ? rho : 0.f;
  }
  float pvv[2] = {0.f, 0.f};
#pragma unroll
  for (int kk = 0; kk < 64; ++kk) {
    const int Ik = kk / 32, kr = kk % 32;
    const int rr = 4 * (kr / 8) + (kr % 4);
    const int hk = (kr / 4) & 1;
    const bool here = (h == hk);
    const float d = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(re[Ik][Ik][rr]), kr + 32 * hk));
    const float pv = __builtin_amdgcn_rcpf(d);
    unsigned ah[2], al[2], bh[2], bl[2];
#pragma unroll
    for (int J = 0; J < 2; ++J) {
      const bool isk = (32 * J + col == kk);
      const float t = (here && !isk) ? pv * 128.f : 0.f;
      const float mb = (here && !isk) ? 0.0078125f : 0.f;
      const float sr = re[Ik][J][rr], si = im[Ik][J][rr];
      split_f16(-sr * t, si * t, ah[J], al[J]);
      split_f16(sr * mb, si * mb, bh[J], bl[J]);
      re[Ik][J][rr] = (here && isk) ? -sr : sr;
    }
#pragma unroll
    for (int I = 0; I < 2; ++I)
#pragma unroll
      for (int J = 0; J < 2; ++J) rank1_split16(re[I][J], im[I][J], ah[I], al[I], bh[J], bl[J]);
#pragma unroll
    for (int J = 0; J < 2; ++J) pvv[J] = (32 * J + col == kk) ? pv : pvv[J];
  }
  gj_unscale_u64(re, im, pvv, post, lane, line);
}

// Mixed-precision Gram for U = 64 (one problem per wave): split half-precision
// H = H_hi + H_lo after a power-of-two scaling, four 32x32 tiles on
// v_mfma_f32_32x32x16_{f16,bf16}; lane l supplies rows 8(l/32) .. 8(l/32)+7 of
// each 16-row chunk at column 32I + l%32 (A) and 32J + l%32 (B).  Then the
// Gauss-Jordan inverse on the matrix cores: FP32 (INV = 0) or split FP16 on
// the normalised Gram (INV = 2).
template <typename HT, int INV, bool FACTOR>
__device__ __forceinline__ c32 gram_inv_mixed_u64(const UlArgs& a, c32 (&A)[64], int lane, int wave,
                                                  float* line, float* stage, float& trg, float* f2) {
  typedef typename HalfMma<HT>::V V;
  const int h = lane >> 5, col = lane & 31;
  const int ls = wave / a.Cp, c = wave % a.Cp;
  const int k = a.blk * a.sc_per_block + ls;
  const bool act = (k < a.n_sc) && (c < a.C);
  const c32* Hk = act ? a.H + (size_t)k * a.B * 64 + (size_t)c * a.S * 64 : a.H;
  const c32* yk = act ? a.y + (size_t)k * a.n_sym * a.B + (size_t)c * a.S : a.y;
  f32x16 re[2][2], im[2][2];
#pragma unroll
  for (int I = 0; I < 2; ++I)
#pragma unroll
    for (int J = 0; J < 2; ++J) {
      re[I][J] = f32x16{};
      im[I][J] = f32x16{};
    }
  // buffer loads over the problem's S rows (as in gram_mfma_u32)
  const __amdgpu_buffer_rsrc_t hrs = __builtin_amdgcn_make_buffer_rsrc(const_cast<c32*>(Hk), 0, act ? a.S * 512 : 0, kBufferWord3);
  const __amdgpu_buffer_rsrc_t yrs = __builtin_amdgcn_make_buffer_rsrc(const_cast<c32*>(yk), 0, act ? a.S * 8 : 0, kBufferWord3);
  // pass 1: scale exponent from the largest |Re|, |Im| (and ||H_c||_F^2 = tr(G_c))
  float mx = 0.f, ss = 0.f;
  for (int s0 = 0; s0 < a.S; s0 += 16) {
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const int s = s0 + 8 * h + t;
      const c32 v0 = __builtin_bit_cast(c32, __builtin_amdgcn_raw_buffer_load_b64(hrs, s * 512 + col * 8, 0, 0));
      const c32 v1 = __builtin_bit_cast(c32, __builtin_amdgcn_raw_buffer_load_b64(hrs, s * 512 + 256 + col * 8, 0, 0));
      mx = fmaxf(mx, fmaxf(fmaxf(fabsf(v0.re), fabsf(v0.im)), fmaxf(fabsf(v1.re), fabsf(v1.im))));
      ss = fmaf(v0.re, v0.re, fmaf(v0.im, v0.im, fmaf(v1.re, v1.re, fmaf(v1.im, v1.im, ss))));
    }
  }
  trg = wave_sum(ss);
  mx = wave_max(mx);
  int x = 0;
  if (mx > 0.f) frexpf(mx, &x);
  const int ex = 14 - x;
  c32 hy0 = cz(), hy1 = cz();
  // pass 2: split and accumulate
  for (int s0 = 0; s0 < a.S; s0 += 16) {
    V rh[2], rl[2], ih[2], il[2], nih[2], nil[2];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const int s = s0 + 8 * h + t;
      const c32 yv = __builtin_bit_cast(c32, __builtin_amdgcn_raw_buffer_load_b64(yrs, s * 8, 0, 0));
#pragma unroll
      for (int I = 0; I < 2; ++I) {
        const c32 v = __builtin_bit_cast(c32, __builtin_amdgcn_raw_buffer_load_b64(hrs, s * 512 + 256 * I + col * 8, 0, 0));
        cmacc(I ? hy1 : hy0, v, yv);
        const float xr = ldexpf(v.re, ex), xi = ldexpf(v.im, ex);
        const HT hr = (HT)xr, hi = (HT)xi;
        rh[I][t] = hr;
        rl[I][t] = (HT)(xr - (float)hr);
        ih[I][t] = hi;
        il[I][t] = (HT)(xi - (float)hi);
        nih[I][t] = -ih[I][t];
        nil[I][t] = -il[I][t];
      }
    }
#pragma unroll
    for (int I = 0; I < 2; ++I)
#pragma unroll
      for (int J = 0; J < 2; ++J) {
        if (INV == 0 && I > J) continue;   // the block inverse does not read it
        re[I][J] = HalfMma<HT>::mma(rh[I], rh[J], re[I][J]);
        re[I][J] = HalfMma<HT>::mma(rh[I], rl[J], re[I][J]);
        re[I][J] = HalfMma<HT>::mma(rl[I], rh[J], re[I][J]);
        re[I][J] = HalfMma<HT>::mma(ih[I], ih[J], re[I][J]);
        re[I][J] = HalfMma<HT>::mma(ih[I], il[J], re[I][J]);
        re[I][J] = HalfMma<HT>::mma(il[I], ih[J], re[I][J]);
        im[I][J] = HalfMma<HT>::mma(rh[I], ih[J], im[I][J]);
        im[I][J] = HalfMma<HT>::mma(rh[I], il[J], im[I][J]);
        im[I][J] = HalfMma<HT>::mma(rl[I], ih[J], im[I][J]);
        im[I][J] = HalfMma<HT>::mma(nih[I], rh[J], im[I][J]);
        im[I][J] = HalfMma<HT>::mma(nih[I], rl[J], im[I][J]);
        im[I][J] = HalfMma<HT>::mma(nil[I], rh[J], im[I][J]);
      }
  }
  const int sh = (INV == 2) ? norm_shift(a.S) : 2 * ex;
#pragma unroll
  for (int I = 0; I < 2; ++I)
#pragma unroll
    for (int J = 0; J < 2; ++J)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        re[I][J][r] = ldexpf(re[I][J][r], -sh);
        im[I][J][r] = ldexpf(im[I][J][r], -sh);
      }
  if (INV == 2)
    gj_invert_split16_u64(re, im, lane, ldexpf(a.rho, 2 * ex - sh), ldexpf(1.f, 2 * ex - sh), line);
  else
    invert_blocks_u64<FACTOR>(re, im, lane, a.rho, line, stage, A, a.cond_max > 0.f ? f2 : nullptr);
  if constexpr (INV == 2) acc_to_rows_u64(re, im, A, h);
  return combine_hy_u64(hy0, hy1, h);
}

// Consensus: every lane of cluster c writes its entry of w_c into its slot;
// after the barrier each lane sums the C clusters of its subcarrier in cluster
// order 1..C (identical sum on every cluster, as if broadcast by the fusion
// node).
// The padding clusters C..Cp-1 of a subcarrier write zeros, so with UNROLL the
// sum runs over all Cp slots (a power of two) with a fully unrolled loop;
// adding the trailing zeros leaves the value unchanged.  Without UNROLL (kernels
// whose register budget the unrolled form would cut into) it is a loop over C.
template <int N>
__device__ __forceinline__ c32 sum_slots(const c32* src, int G) {
  c32 w = src[0];
#pragma unroll
  for (int cc = 1; cc < N; ++cc) w = cadd(w, src[cc * G]);
  return w;
}

// Sum of a complex value over the P = 64 / G lane groups of a wave (lanes l,
// l ^ G, l ^ 2G, ...), the same bits on every lane: pairs of groups first,
// then pairs of pairs.  The real and imaginary parts travel together: one
// v_permlane16_swap of (re, im) leaves the pair sums of re on the even and of
// im on the odd rows of 16 lanes, one v_permlane32_swap adds the halves, and a
// last swap hands every lane both components.
template <int P>
__device__ __forceinline__ c32 wave_group_sum(c32 w) {
  if constexpr (P >= 8) w = c32{pair_sum<8>(w.re), pair_sum<8>(w.im)};
  if constexpr (P >= 4) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(w.re), __float_as_uint(w.im), false, false);
    const float s = __uint_as_float(a[0]) + __uint_as_float(a[1]);   // rows: re01 im01 re23 im23
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(s), __float_as_uint(s), false, false);
    const float t = __uint_as_float(b[0]) + __uint_as_float(b[1]);   // rows: re im re im (totals)
    const auto c = __builtin_amdgcn_permlane16_swap(__float_as_uint(t), __float_as_uint(t), false, false);
    return c32{__uint_as_float(c[0]), __uint_as_float(c[1])};
  } else {
    const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(w.re), __float_as_uint(w.im), false, false);
    const float s = __uint_as_float(a[0]) + __uint_as_float(a[1]);   // halves: re | im
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(s), __float_as_uint(s), false, false);
    return c32{__uint_as_float(b[0]), __uint_as_float(b[1])};
  }
}

template <bool UNROLL = true>
__device__ __forceinline__ c32 consensus(c32 wc, int buf, int ls, int G, int u, int C, int Cp, const Smem& sm,
                                         int slot, int nw) {
  c32* cb = sm.cons + buf * nw * 64;
  cb[slot] = wc;
  __syncthreads();
  const c32* src = cb + (size_t)ls * Cp * G + u;
  if (!UNROLL) {
    c32 w = cz();
    for (int cc = 0; cc < C; ++cc) w = cadd(w, src[cc * G]);
    return w;
  }
  switch (Cp) {
    case 1: return src[0];
    case 2: return sum_slots<2>(src, G);
    case 4: return sum_slots<4>(src, G);
    case 8: return sum_slots<8>(src, G);
    default: return sum_slots<16>(src, G);
  }
}

// The consensus of the lane-group layout with P = 64 / G problems per wave.
// When the padded cluster count Cp is at least P, the wave's P problems are
// clusters P j .. P j + P - 1 of one subcarrier: their vectors are summed in
// registers first (pairs of lanes l, l ^ G, then l, l ^ 2G, ...: the same
// tree on every lane, so every lane holds the same bits), and only the
// first group of each wave writes its slot; the readers then add Cp / P
// slots in cluster order.  Otherwise, as consensus().
template <int G>
__device__ __forceinline__ c32 consensus_w(c32 wc, int buf, int ls, int u, int g, int C, int Cp, const Smem& sm,
                                           int slot, int nw) {
  constexpr int P = 64 / G;
  if constexpr (P == 1) {
    (void)g;
    return consensus<true>(wc, buf, ls, G, u, C, Cp, sm, slot, nw);
  } else {
    if (Cp < P) return consensus<true>(wc, buf, ls, G, u, C, Cp, sm, slot, nw);
    const c32 w = wave_group_sum<P>(wc);
    c32* cb = sm.cons + buf * nw * 64;
    if (g == 0) cb[slot] = w;
    __syncthreads();
    const c32* src = cb + (size_t)ls * Cp * G + u;
    switch (Cp / P) {
      case 1: return src[0];
      case 2: return sum_slots<2>(src, P * G);
      case 4: return sum_slots<4>(src, P * G);
      default: return sum_slots<8>(src, P * G);
    }
  }
}

// ---------------------------------------------------------------------------
// Several received vectors over one channel (U = 16, 32, 64): eight symbols at a
// time as the 16 columns (eight real, eight imaginary parts) of 16 x 16 x 4
// products.  A complex product M X is Re M [Xr | Xi] + Im M [-Xi | Xr], the
// second operand a rotation of the first by eight lanes.  Rows 4 q + r of a
// column block sit in register r of lane group q, both as an accumulator and as
// the operand of step r, so the vectors pass from product to product without
// moving, and the eight symbols share each barrier of the consensus.
// Bound by the issue of the products: the vector units need 128 multiply-adds per
// symbol, product and wave at U = 32 (512 cycles), these 64 instructions of 32
// cycles for eight symbols (256 cycles each).  Measured, 9536 subcarriers at
// B = 256, U = 32, C = 8, T = 5: seven symbols 783 -> 544 us, fourteen 1370 -> 852.
// Registers: U = 32 capped at 168 (three waves per SIMD; 169 and two: 626 us for
// seven symbols), U = 16 at 128.  Against stored factors (the same sizes) seven
// symbols 687 -> 370 us and fourteen 1288 -> 677.
// ---------------------------------------------------------------------------

// [Xr | Xi] -> [Xi | Xr], the first half times sg and the second times -sg (the
// sign is the lane's)
__device__ __forceinline__ float swap_parts(float x, float sg) {
  return sg * __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x128, 0xF, 0xF, true));
}

// H_c^H y_c of symbols n0 .. n0 + 7 for the problems of the wave (zero past n_sym).
// H16: H from the packed FP16 channel, widened, the tile's power-of-two scale
// applied at the end (exact).
template <int G, bool H16>
__device__ __forceinline__ void syms_hy(const UlArgs& a, int n0, f32x4 (&hy)[64 / G][G / 16], int lane, int wave) {
  constexpr int P = 64 / G, NT = G / 16;
  const int q = lane >> 4, col = lane & 15, j = col & 7;
  const float sg = (col & 8) ? -1.f : 1.f;   // conj(H): [yi | -yr]
  __amdgpu_buffer_rsrc_t hrs[P], yrs[P];
  f32x4 hi[P][NT];
  const int nj = min(8, a.n_sym - n0);
#pragma unroll
  for (int p = 0; p < P; ++p) {
    const int lp = wave * P + p;
    const int ls = lp / a.Cp, c = lp % a.Cp;
    const int k = a.blk * a.sc_per_block + ls;
    const bool act = (k < a.n_sc) && (c < a.C);
    const size_t ho = act ? (size_t)k * a.B * G + (size_t)c * a.S * G : 0;
    const c32* yp = act ? a.y + ((size_t)k * a.n_sym + n0) * a.B + (size_t)c * a.S : a.y;
    if constexpr (H16)
      hrs[p] = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(a.H16 + ho), 0, act ? a.S * G * 4 : 0, kBufferWord3);
    else
      hrs[p] = __builtin_amdgcn_make_buffer_rsrc(const_cast<c32*>(a.H + ho), 0, act ? a.S * G * 8 : 0, kBufferWord3);
    yrs[p] = __builtin_amdgcn_make_buffer_rsrc(const_cast<c32*>(yp), 0, act ? ((nj - 1) * a.B + a.S) * 8 : 0, kBufferWord3);
#pragma unroll
    for (int t = 0; t < NT; ++t) hy[p][t] = hi[p][t] = f32x4{};
  }
  struct Rows {
    std::conditional_t<H16, uint32_t, c32> h[P][NT];
    float y[P];
  };
  auto fetch = [&](int s0, Rows& d) {
    const int s = s0 + q;
    // (an offset past the range for rows past S and symbols past n_sym: zero)
    const unsigned yo = (s < a.S && j < nj) ? (unsigned)(j * a.B + s) * 8u + ((col & 8) ? 4u : 0u) : 0x80000000u;
#pragma unroll
    for (int p = 0; p < P; ++p) {
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        if constexpr (H16)
          d.h[p][t] = __builtin_amdgcn_raw_buffer_load_b32(hrs[p], s * (G * 4) + t * 64 + col * 4, 0, 0);
        else
          d.h[p][t] = __builtin_bit_cast(
              c32, __builtin_amdgcn_raw_buffer_load_b64(hrs[p], s * (G * 8) + t * 128 + col * 8, 0, 0));
      }
      d.y[p] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(yrs[p], yo, 0, 0));
    }
  };
  auto accumulate = [&](const Rows& d) {
#pragma unroll
    for (int p = 0; p < P; ++p) {
      const float ys = swap_parts(d.y[p], sg);
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        c32 h;
        if constexpr (H16) h = widen_h16(d.h[p][t]);
        else h = d.h[p][t];
        hy[p][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(h.re, d.y[p], hy[p][t], 0, 0, 0);
        hi[p][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(h.im, ys, hi[p][t], 0, 0, 0);
      }
    }
  };
  Rows d0, d1;
  fetch(0, d0);
  fetch(4, d1);
  int s0 = 0;
  for (; s0 + 4 < a.S; s0 += 8) {
    accumulate(d0);
    fetch(s0 + 8, d0);
    accumulate(d1);
    fetch(s0 + 12, d1);
  }
  if (s0 < a.S) accumulate(d0);
#pragma unroll
  for (int p = 0; p < P; ++p) {
    float scale = 1.f;
    if constexpr (H16) {
      const int lp = wave * P + p;
      const int ls = lp / a.Cp, c = lp % a.Cp;
      const int k = a.blk * a.sc_per_block + ls;
      scale = (k < a.n_sc && c < a.C) ? a.hscale[(size_t)k * a.C + c] : 0.f;
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      hy[p][t] += hi[p][t];
      if constexpr (H16) hy[p][t] *= scale;
    }
  }
}

// The rows of the lane layout (lane 16 g + i: row i of lane group g) as operands:
// A[16 J + 4 g + s] of lane 16 q + i becomes entry (i, 16 J + 4 q + s) of group g.
template <int G>
__device__ __forceinline__ void rows_to_operands(c32 (&A)[G]) {
#pragma unroll
  for (int J = 0; J < G / 16; ++J)
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      float re[4], im[4];
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        re[m] = A[16 * J + 4 * m + s].re;
        im[m] = A[16 * J + 4 * m + s].im;
      }
      transpose_groups(re);
      transpose_groups(im);
#pragma unroll
      for (int g = 0; g < 4; ++g) A[16 * J + 4 * g + s] = c32{re[g], im[g]};
    }
}

// B^{-1} x of problem p of the wave.  BLOCK: the block factors of gram_blocks_u32
// and invert_blocks_u64 (their conjugates), else the whole inverse.  The products
// with the real and the imaginary parts have accumulators of their own: shorter
// sums, and two chains in flight per row block.
template <int G, bool BLOCK>
__device__ __forceinline__ void syms_matvec(const c32 (&A)[G], int p, const f32x4 (&x)[G / 16], f32x4 (&out)[G / 16],
                                            float sg) {
  constexpr int NT = G / 16, NH = BLOCK ? NT / 2 : NT;
  // acc[I] = sum of column blocks J0 .. J0 + NH - 1 times v[J - J0]
  auto mul = [&](int J0, const f32x4 (&v)[NH], f32x4 (&acc)[NT]) {
    f32x4 im[NT];
#pragma unroll
    for (int I = 0; I < NT; ++I) acc[I] = im[I] = f32x4{};
#pragma unroll
    for (int J = 0; J < NH; ++J)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float w = swap_parts(v[J][r], sg);
#pragma unroll
        for (int I = 0; I < NT; ++I) {
          const c32 m = A[16 * (J0 + J) + 4 * (p * NT + I) + r];
          acc[I] = __builtin_amdgcn_mfma_f32_16x16x4f32(m.re, v[J][r], acc[I], 0, 0, 0);
          im[I] = __builtin_amdgcn_mfma_f32_16x16x4f32(m.im, w, im[I], 0, 0, 0);
        }
      }
#pragma unroll
    for (int I = 0; I < NT; ++I) acc[I] += im[I];
  };
  if constexpr (!BLOCK) {
    mul(0, x, out);
  } else {
    f32x4 v[NH], b[NT];
#pragma unroll
    for (int J = 0; J < NH; ++J) v[J] = x[J];
    mul(0, v, out);                                       // Pi q_1 | W^H q_1
#pragma unroll
    for (int J = 0; J < NH; ++J) v[J] = x[NH + J] - out[NH + J];   // t
    mul(NH, v, b);                                        // X t | Si t
#pragma unroll
    for (int J = 0; J < NH; ++J) {
      out[J] = out[J] - b[J];
      out[NH + J] = b[NH + J];
    }
  }
}

// Sum of w over the wps waves of a subcarrier through their stage buffers, in
// cluster order.
template <int G>
__device__ __forceinline__ void syms_consensus(f32x4 (&w)[G / 16], float4* cons, int& buf, int lane, int wave, int wps) {
  constexpr int NT = G / 16, pitch = kStageWave / 2;
  constexpr bool TWO = 2 * NT * 64 <= pitch;   // two buffers in turn (U = 64: one, and a second barrier)
  if (!TWO) __syncthreads();
  float4* mine = cons + wave * pitch + buf * NT * 64 + lane;
#pragma unroll
  for (int t = 0; t < NT; ++t) mine[t * 64] = make_float4(w[t][0], w[t][1], w[t][2], w[t][3]);
  __syncthreads();
  const float4* src = cons + wave / wps * wps * pitch + buf * NT * 64 + lane;
  for (int i = 0; i < wps; ++i)
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const float4 v = src[i * pitch + t * 64];
      if (i == 0) w[t] = f32x4{v.x, v.y, v.z, v.w};
      else w[t] += f32x4{v.x, v.y, v.z, v.w};
    }
  if (TWO) buf ^= 1;
}

// Outputs of symbols n0 .. n0 + 7 of subcarrier k: the pair of lanes with a
// symbol's real and imaginary parts shares its users, two each of the four.
// Returns the lane's status bits.
template <int G>
__device__ __forceinline__ int syms_store(const UlArgs& a, const f32x4 (&s)[G / 16], int k, int n0, int lane, float guard) {
  const int im = (lane >> 3) & 1, n = n0 + (lane & 7);
  int fl = 0;
#pragma unroll
  for (int t = 0; t < G / 16; ++t) {
    float o[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) o[r] = swap_parts(s[t][r], 1.f);
    const c32 e0 = im ? c32{o[2], s[t][2]} : c32{s[t][0], o[0]};
    const c32 e1 = im ? c32{o[3], s[t][3]} : c32{s[t][1], o[1]};
    if (n < a.n_sym) {
      const size_t at = ((size_t)k * a.n_sym + n) * G + 16 * t + 4 * (lane >> 4) + 2 * im;
      a.shat[at] = e0;
      a.shat[at + 1] = e1;
      if (a.hard) {
        a.hard[at] = (uint8_t)(slice_dim(e0.re, a.kappa, a.L) + a.L * slice_dim(e0.im, a.kappa, a.L));
        a.hard[at + 1] = (uint8_t)(slice_dim(e1.re, a.kappa, a.L) + a.L * slice_dim(e1.im, a.kappa, a.L));
        if (near_threshold(e0.re, a.kappa, a.L, guard) || near_threshold(e0.im, a.kappa, a.L, guard) ||
            near_threshold(e1.re, a.kappa, a.L, guard) || near_threshold(e1.im, a.kappa, a.L, guard))
          fl |= 2;
      }
      if (nonfinite(e0) || nonfinite(e1)) fl |= 1;
    }
  }
  return fl;
}

// The subcarrier's status word from the bits of its first wave.
__device__ __forceinline__ void syms_flags(const UlArgs& a, int fl, int k, bool first, int lane) {
  if (!a.flags) return;
  const int bits = group_flags<64>(fl, 0);
  if (first && lane == 0 && k < a.n_sc) {
    a.flags[k] = bits;
    if ((bits & kStatusReslice) && a.any) *a.any = a.epoch;
  }
}

// The iterations of all symbols.  A: the factors as operands; cons: the waves'
// stage buffers.  All problems of a wave belong to one subcarrier (Cp >= 64 / G).
// Returns the status bits of the wave's outputs.
template <int G, bool BLOCK, bool H16>
__device__ __forceinline__ int syms_iterate(const UlArgs& a, const c32 (&A)[G], int lane, int wave, float4* cons,
                                            float guard) {
  constexpr int P = 64 / G, NT = G / 16;
  const float sg = ((lane & 8) != 0) == BLOCK ? -1.f : 1.f;   // [-xi | xr], or with conjugated factors [xi | -xr]
  const int wps = a.Cp / P;                           // waves of a subcarrier
  const int w0 = wave / wps * wps;                    // the first of them
  const int k = a.blk * a.sc_per_block + wave / wps;
  int fl = 0, buf = 0;
  bool act[P];
#pragma unroll
  for (int p = 0; p < P; ++p) act[p] = k < a.n_sc && (wave - w0) * P + p < a.C;
  for (int n0 = 0; n0 < a.n_sym; n0 += 8) {
    f32x4 z[P][NT], lam[P][NT], yreg[P][NT], s[NT];
    {
      f32x4 hy[P][NT];
      syms_hy<G, H16>(a, n0, hy, lane, wave);
#pragma unroll
      for (int p = 0; p < P; ++p) syms_matvec<G, BLOCK>(A, p, hy[p], yreg[p], sg);
    }
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        z[p][t] = yreg[p][t];
        lam[p][t] = f32x4{};
      }
    // sum over the clusters of z + lambda: the wave's problems in registers, the
    // waves through LDS, in cluster order; then the s-update
    auto consensus_s = [&]() {
      f32x4 w[NT];
#pragma unroll
      for (int t = 0; t < NT; ++t) w[t] = f32x4{};
#pragma unroll
      for (int p = 0; p < P; ++p) {
        if (act[p]) {
#pragma unroll
          for (int t = 0; t < NT; ++t) w[t] += z[p][t] + lam[p][t];
        }
      }
      syms_consensus<G>(w, cons, buf, lane, wave, wps);
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          s[t][r] = (a.reg == 2) ? fminf(fmaxf(w[t][r] * a.invC, -a.box_r), a.box_r) : w[t][r] * a.inv_den;
    };
    consensus_s();
    for (int it = 2; it <= a.T; ++it) {
#pragma unroll
      for (int p = 0; p < P; ++p) {
        f32x4 q[NT], bq[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            lam[p][t][r] = fmaf(a.gamma, z[p][t][r] - s[t][r], lam[p][t][r]);
            q[t][r] = s[t][r] - lam[p][t][r];
          }
        syms_matvec<G, BLOCK>(A, p, q, bq, sg);
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
          for (int r = 0; r < 4; ++r) z[p][t][r] = fmaf(a.rho, bq[t][r], yreg[p][t][r]);
      }
      consensus_s();
    }
    if (wave == w0 && k < a.n_sc) fl |= syms_store<G>(a, s, k, n0, lane, guard);
  }
  return fl;
}

// ---------------------------------------------------------------------------
// Algorithm 1, U x U branch (S >= U), FP32.  Group size G = U.
// ---------------------------------------------------------------------------
// HALF: 0 FP32 Gram, 1 / 2 split FP16 / BF16 Gram (mixed modes, U = 32, 64).
// INV (mixed modes): 0 FP32 matrix-core inverse, 1 FP64 VALU inverse (U = 32),
// 2 split-FP16 matrix-core inverse.
// STAGE: 0 preprocessing and iterations; 1 preprocessing only, B_c^{-1} is
// written to a.fac (a static channel factored once); 2 iterations only, B_c^{-1}
// read from a.fac (every symbol's H_c^H y_c by the VALU pass); 3 as 2 with H
// read from the packed FP16 channel; 4 (U = 32, FP32) as 1, and H also
// written as the packed FP16 channel in the same launch.
// LINE: the block factors' products at U = 32 through the broadcast line
// (block_matvec) instead of row broadcasts (block_matvec_u32).
template <int G, int HALF, int INV, int STAGE, bool SYMS, bool LINE>
__device__ __forceinline__ void admm_ul_body(const UlArgs& a);

// Registers: at U = 64 three waves per SIMD (168; two with 171: C = 3, T = 40, 600
// subcarriers 155 us against 123).
template <int G, int HALF, int INV, int STAGE, bool SYMS = false, bool LINE = false>
__global__ void __launch_bounds__(512, !SYMS ? (G == 64 && HALF == 0 && STAGE == 0 ? 3 : LINE ? 4 : 1) : G == 16 ? 4 : G == 32 ? 3 : 2) admm_ul_f32(UlArgs a) {
  a.blk = blockIdx.x;
  admm_ul_body<G, HALF, INV, STAGE, SYMS, LINE>(a);
}

// Several frames of the same U in one launch (FP32, one-shot): frame f owns the
// workgroups first[f] .. first[f+1]-1, in its own launch plan (all frames share
// the waves per workgroup).  A workgroup counts the frames that start at or
// before it (first[] past the last frame holds INT_MAX), so the loads of first[]
// are in flight together.  The frames' argument blocks travel in the kernel
// arguments.  One block of subcarriers per workgroup: with a persistent grid
// (1024 workgroups in a loop over the blocks) eight uneven U = 16 frames took
// 57 us instead of 55, the loop's registers costing a wave per SIMD.
// SYMS: some frame takes the column form of the iterations (symbol_columns).  One
// launch for both forms, though the columns' registers cost the other frames a wave
// per SIMD: eight frames, one of them of seven symbols (us, one launch | one per
// form): U = 16, 12 subcarriers each 38 | 44, 1200 each 90 | 98; U = 32, 100 each
// 50 | 63, 1200 each 356 | 340; U = 64, 12 each 82 | 135, 300 each 556 | 635.
template <int G, bool SYMS, bool LINE = false>
__global__ void __launch_bounds__(512, !SYMS ? (G == 64 ? 3 : LINE ? 4 : 1) : G == 16 ? 4 : G == 32 ? 3 : 2) admm_ul_f32_batch(UlBatch b) {
  const int vb = blockIdx.x;
  int f = 0;
#pragma unroll
  for (int i = 1; i < kMaxBatch; ++i) f += (b.first[i] <= vb) ? 1 : 0;
  UlArgs a = b.f[f];
  a.blk = vb - b.first[f];
  if constexpr (SYMS) {
    if (symbol_columns(G, a.n_sym, a.B, a.S, a.C, a.T)) return admm_ul_body<G, 0, 0, 0, true, false>(a);
  }
  admm_ul_body<G, 0, 0, 0, false, LINE>(a);
}

template <int G, int HALF, int INV, int STAGE, bool SYMS, bool LINE>
__device__ __forceinline__ void admm_ul_body(const UlArgs& a) {
  constexpr int P = 64 / G;
  constexpr bool RESIDENT = (STAGE == 2 || STAGE == 3);   // iterations against stored factors
  constexpr bool FACTOR = (STAGE == 1 || STAGE == 4);     // preprocessing only
  constexpr bool BLOCKS = (G == 32 && HALF == 0 && STAGE == 0);   // the inverse as 16 x 16 block factors
  constexpr bool BLOCKS64 = (G == 64 && INV == 0 && STAGE == 0);  // the same with 32 x 32 blocks
  extern __shared__ float4 smem_raw[];
  const int nw = blockDim.x >> 6;
  Smem sm = carve(reinterpret_cast<c32*>(smem_raw), nw);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave-uniform: addresses in SALU
  const int g = lane / G, u = lane % G;
  const int lp = wave * P + g;
  const int ls = lp / a.Cp, c = lp % a.Cp;
  const int k = a.blk * a.sc_per_block + ls;
  const bool active = (k < a.n_sc) && (c < a.C);
  const int slot = wave * 64 + lane;
  c32* line = sm.line + wave * 64;
  const int gbase = g * G;

  // Preprocessing (Alg. 1, S > U branch): B_c = H_c^H H_c + rho I, B_c^{-1}.
  c32 A[G];
  // (the U = 16 Gram and the U = 32 factor staging write every entry of every
  // lane's row: no clearing)
  if constexpr (!(G == 16 && !RESIDENT) && !(G == 32 && RESIDENT) && !BLOCKS && !BLOCKS64) {
#pragma unroll
    for (int v = 0; v < G; ++v) A[v] = cz();
  }
  c32 hy0 = cz();
  float trg = 0.f;   // tr(G_c) (mixed modes)
  float f2b = 0.f;   // ||B_c^{-1}||_F^2 (mixed modes, block factors, FP64 factor rule)
  // U = 16, FP32, iterations in the same launch: the inverse keeps its lazy
  // scales (B^{-1} = 2 D - D S D, D = diag(pv): off the diagonal
  // -S_uv pv_u pv_v), which every product applies to its operand and result
  // instead of to the U x U entries.
  constexpr bool LAZY = (G == 16 && HALF == 0 && STAGE == 0);
  float pvl = 1.f;
  auto bmat = [&](c32 q) -> c32 {
    if constexpr (LAZY) {
      // (the sweeps leave the diagonal un-negated: + 2 pv_u q_u)
      const c32 r = group_matvec<G>(A, cscale(q, pvl), u, line, gbase);
      const float tp = 2.f * pvl;
      return c32{fmaf(tp, q.re, -pvl * r.re), fmaf(tp, q.im, -pvl * r.im)};
    } else if constexpr (BLOCKS) {
      if constexpr (LINE) return block_matvec<G>(A, q, line, gbase, lane, (lane & 16) == 0);
      else return block_matvec_u32(A, q, (lane & 16) == 0);
    } else if constexpr (BLOCKS64) {
      return block_matvec<G>(A, q, line, gbase, lane, lane < 32);
    } else {
      return group_matvec<G>(A, q, u, line, gbase);
    }
  };
  // Resident factors of this problem: B_c^{-1} is Hermitian, so only its
  // upper triangle is stored, column by column (entry (i, v), i <= v, at
  // v (v + 1) / 2 + i; G (G + 1) / 2 values per problem).  Lane u's row
  // takes entry v from column v (v >= u) or, conjugated, from column u
  // (v < u): one load per entry, coalesced over the lanes of the first kind.
  constexpr int NT = G * (G + 1) / 2;
  const size_t fo = ((size_t)k * a.C + c) * NT;
  if constexpr (RESIDENT && G == 32) {
    // The lanes of the other kind would read 32 different cache lines per
    // load, so each problem's triangle (NT = 528 values, the size of the
    // wave's stage buffer) first goes through LDS with 16-byte coalesced
    // loads, one problem of the wave at a time.  Both candidate entries are
    // inside the triangle for every (u, v) (indices at most NT - 1), so each
    // lane reads both and keeps one.
    // Both problems' factor loads are issued first, and symbol 0's
    // H_c^H y_c is formed while they are in flight.
    c32* tri = sm.stage + wave * kStageWave;
    const int csu = u * (u + 1) / 2;
    constexpr int NQ = (NT / 2 + 63) / 64;
    float4 tq[P][NQ];
    bool tv[P];
#pragma unroll
    for (int pp = 0; pp < P; ++pp) {
      const int lq = wave * P + pp;
      const int kq = a.blk * a.sc_per_block + lq / a.Cp, cq = lq % a.Cp;
      tv[pp] = kq < a.n_sc && cq < a.C;
      // a buffer load over the problem's NT entries (none when inactive):
      // the range check zeroes the slots past the triangle without selects
      const __amdgpu_buffer_rsrc_t frs = __builtin_amdgcn_make_buffer_rsrc(
          const_cast<c32*>(a.fac + (tv[pp] ? ((size_t)kq * a.C + cq) * NT : 0)), 0, tv[pp] ? NT * 8 : 0, kBufferWord3);
#pragma unroll
      for (int i = 0; i < NQ; ++i)
        tq[pp][i] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(frs, (i * 64 + lane) * 16, 0, 0));
    }
    if constexpr (SYMS)
      (void)hy0;
    else if constexpr (STAGE == 3)
      hy0 = cluster_hy_direct<G, true>(a, k, c, 0, u, active);
    else
      hy0 = cluster_pass<G, false>(a.H, a.y, A, k, c, 0, u, g, lane, wave, active, a.B, a.S, G, a.n_sym, sm);
#pragma unroll
    for (int pp = 0; pp < P; ++pp) {
      if (tv[pp]) {
        float4* dst = reinterpret_cast<float4*>(tri);
#pragma unroll
        for (int i = 0; i < NQ; ++i)
          if (i * 64 + lane < NT / 2) dst[i * 64 + lane] = tq[pp][i];
      }
      wave_lds_sync();
      // (an inactive problem reads whatever the buffer holds; its results
      // are never stored)
      if (g == pp) {
#pragma unroll
        for (int v = 0; v < G; ++v) {
          const c32 e1 = tri[v * (v + 1) / 2 + u];   // entry (u, v), v >= u
          const c32 e2 = tri[csu + v];               // entry (v, u), v < u
          A[v] = (v >= u) ? e1 : c32{e2.re, -e2.im};
        }
      }
      wave_lds_sync();
    }
  } else if constexpr (RESIDENT) {
    if (active) {
      const int csu = u * (u + 1) / 2;
#pragma unroll
      for (int v = 0; v < G; ++v) {
        const bool up = v >= u;
        const c32 e = a.fac[fo + (up ? (size_t)(v * (v + 1) / 2 + u) : (size_t)(csu + v))];
        A[v] = up ? e : c32{e.re, -e.im};
      }
    }
  } else if constexpr (BLOCKS) {
    hy0 = gram_blocks_u32(a, A, lane, wave, reinterpret_cast<float*>(sm.stage + wave * kStageWave));
  } else if constexpr (G == 32 && HALF == 0) {
    hy0 = gram_mfma_u32<true, STAGE == 4>(a, A, lane, wave, reinterpret_cast<float*>(line),
                                          reinterpret_cast<float*>(sm.stage + wave * kStageWave));
  } else if constexpr (G == 32 && HALF == 1) {
    hy0 = gram_inv_mixed_u32<_Float16, INV>(a, A, lane, wave, reinterpret_cast<c64*>(sm.stage + wave * kStageWave),
                                            trg);
  } else if constexpr (G == 32 && HALF == 2) {
    hy0 = gram_inv_mixed_u32<__bf16, INV>(a, A, lane, wave, reinterpret_cast<c64*>(sm.stage + wave * kStageWave),
                                          trg);
  } else if constexpr (G == 16) {
    if constexpr (LAZY) {
      hy0 = gram_mfma_u16<true, true>(a, A, lane, wave, sm.stage + wave * kStageWave, &pvl);
    } else {
      hy0 = gram_mfma_u16<true>(a, A, lane, wave, sm.stage + wave * kStageWave);
      gj_invert<G>(A, u, line, gbase);
    }
  } else if constexpr (G == 64 && HALF == 0) {
    hy0 = gram_mfma_u64<FACTOR ? 2 : 1>(a, A, lane, wave, reinterpret_cast<float*>(line),
                              reinterpret_cast<float*>(sm.stage + wave * kStageWave));
  } else if constexpr (G == 64 && HALF == 1) {
    hy0 = gram_inv_mixed_u64<_Float16, INV, FACTOR>(a, A, lane, wave, reinterpret_cast<float*>(line),
                                            reinterpret_cast<float*>(sm.stage + wave * kStageWave), trg, &f2b);
  } else if constexpr (G == 64 && HALF == 2) {
    hy0 = gram_inv_mixed_u64<__bf16, INV, FACTOR>(a, A, lane, wave, reinterpret_cast<float*>(line),
                                          reinterpret_cast<float*>(sm.stage + wave * kStageWave), trg, &f2b);
  } else {
    hy0 = cluster_pass<G, true>(a.H, a.y, A, k, c, 0, u, g, lane, wave, active, a.B, a.S, G, a.n_sym, sm);
#pragma unroll
    for (int v = 0; v < G; ++v)
      if (v == u) A[v].re += a.rho;
    gj_invert<G>(A, u, line, gbase);
  }
  if constexpr (FACTOR && G == 32) {
    // Through the wave's stage buffer, one problem at a time, then 16-byte
    // coalesced stores.  Lane u writes entry v of its row to v (v + 1) / 2 + u
    // for every v in increasing order: for v >= u that is entry (u, v) of the
    // triangle; for v < u the position belongs to a later column w > v, whose
    // own write (step w, lane u') comes after it and replaces it.  Every
    // position is inside the triangle (at most NT - 1).
    c32* tri = sm.stage + wave * kStageWave;
#pragma unroll
    for (int pp = 0; pp < P; ++pp) {
      if (g == pp) {
#pragma unroll
        for (int v = 0; v < G; ++v) tri[v * (v + 1) / 2 + u] = A[v];
      }
      wave_lds_sync();
      const int lq = wave * P + pp;
      const int kq = a.blk * a.sc_per_block + lq / a.Cp, cq = lq % a.Cp;
      if (kq < a.n_sc && cq < a.C) {
        float4* dst = reinterpret_cast<float4*>(a.fac + ((size_t)kq * a.C + cq) * NT);
        const float4* src = reinterpret_cast<const float4*>(tri);
#pragma unroll
        for (int i = 0; i < (NT / 2 + 63) / 64; ++i)
          if (i * 64 + lane < NT / 2) dst[i * 64 + lane] = src[i * 64 + lane];
      }
      wave_lds_sync();
    }
    return;
  } else if constexpr (FACTOR) {
    if (active) {
#pragma unroll
      for (int v = 0; v < G; ++v)
        if (v >= u) a.fac[fo + (size_t)(v * (v + 1) / 2 + u)] = A[v];
    }
    return;
  }

  // FP64 factor rule (mixed modes, FP32 inverse): kappa_hat = tr(B_c)
  // ||B_c^{-1}||_F bounds the condition number kappa_2(B_c) from above (the
  // largest eigenvalue is at most the trace, and ||B_c^{-1}||_2 at most the
  // Frobenius norm).  A subcarrier with a cluster above cond_max goes to the
  // FP64 pass.  Below it the FP32 error grows in proportion to the
  // conditioning, so the re-slice guard is widened by kappa_hat / cond_ref
  // (cond_ref: the largest kappa_hat of the channels the guard was measured
  // on).  Each problem's kappa_hat reaches the output lanes of cluster 0
  // through one LDS slot, read after the first consensus barrier.
  constexpr bool COND = (HALF > 0 && INV == 0 && STAGE == 0);
  float* cond_slot = reinterpret_cast<float*>(sm.aux);
  float guard = a.guard;
  if constexpr (COND) {
    if (a.cond_max != 0.f) {
      float f2 = f2b;
      if constexpr (!BLOCKS64) {
#pragma unroll
        for (int v = 0; v < G; ++v) f2 = fmaf(A[v].re, A[v].re, fmaf(A[v].im, A[v].im, f2));
        f2 = group_sum<G>(f2);
      }
      const float kh = (trg + (float)G * a.rho) * sqrtf(f2);
      if (u == 0) cond_slot[ls * a.Cp + c] = active ? kh : 0.f;
    }
  }

  if constexpr (SYMS) {
    const int lead = wave * P;   // the wave's first problem
    const int kw = a.blk * a.sc_per_block + lead / a.Cp;
    int fl = 0;
    if constexpr (COND) {
      if (a.cond_max != 0.f) {
        __syncthreads();
        const float* kc = cond_slot + lead / a.Cp * a.Cp;
        float km = 0.f;
        bool bad = a.cond_max < 0.f;
        for (int cc = 0; cc < a.C; ++cc) {
          bad = bad || !(kc[cc] <= a.cond_max);   // NaN and infinity fail the comparison
          km = fmaxf(km, kc[cc]);
        }
        if (bad) fl |= kStatusReslice | kStatusIllcond;
        guard = a.guard * fmaxf(1.f, km / a.cond_ref);
      }
    }
    if constexpr (LAZY) {
      // 2 D - D S D, each entry rounded once (the scales' product as a pair, of
      // their mantissas: the powers of two go to the entry, which they bring to
      // the size of the result)
      const float ml = __builtin_amdgcn_frexp_mantf(pvl);
      const int el = __builtin_amdgcn_frexp_expf(pvl);
      static_for<16>([&](auto vc) {
        constexpr int v = decltype(vc)::value;
        const float mv = bcast16<v>(ml);
        const int ev = el + __builtin_amdgcn_mov_dpp(el, 0x150 + v, 0xF, 0xF, true);
        const float hi = -ml * mv, lo = fmaf(-ml, mv, -hi);
        const c32 s = cldexp(A[v], ev);
        A[v] = c32{fmaf(hi, s.re, fmaf(lo, s.re, u == v ? 2.f * pvl : 0.f)), fmaf(hi, s.im, lo * s.im)};
      });
    }
    rows_to_operands<G>(A);
    fl |= syms_iterate<G, BLOCKS || BLOCKS64, STAGE == 3>(a, A, lane, wave, reinterpret_cast<float4*>(sm.stage), guard);
    syms_flags(a, fl, kw, lead % a.Cp == 0, lane);
    return;
  }

  int buf = 0;
  int fl = 0;   // status bits of this lane's outputs (bit 0 non-finite, bit 1 re-slice, bit 2 ill-conditioned)
  for (int n = 0; n < a.n_sym; ++n) {
    c32 hy = hy0;
    // (with U = 32 factors, symbol 0's H_c^H y_c was formed with the factor loads)
    constexpr bool HY0 = (RESIDENT && G == 32);
    if constexpr (STAGE == 3) {
      if (!HY0 || n > 0) hy = cluster_hy_direct<G, true>(a, k, c, n, u, active);
    } else if (n > 0 || (STAGE == 2 && !HY0)) {
      hy = cluster_pass<G, false, G == 64 && STAGE == 0>(a.H, a.y, A, k, c, n, u, g, lane, wave, active, a.B, a.S, G,
                                                         a.n_sym, sm);
    }
    // y_c^reg = B_c^{-1} H_c^H y_c; z = y^reg; lambda = 0
    const c32 yreg = bmat(hy);
    c32 z = yreg, lam = cz();
    c32 w = (HALF == 0) ? consensus_w<G>(active ? z : cz(), buf, ls, u, g, a.C, a.Cp, sm, slot, nw)
                        : consensus<false>(active ? z : cz(), buf, ls, G, u, a.C, a.Cp, sm, slot, nw);
    buf ^= 1;
    if constexpr (COND) {
      // the barrier inside the consensus above has made every cluster's estimate visible
      if (n == 0 && a.cond_max != 0.f && c == 0) {
        float km = 0.f;
        bool bad = a.cond_max < 0.f;
        for (int cc = 0; cc < a.C; ++cc) {
          const float kc = cond_slot[ls * a.Cp + cc];
          bad = bad || !(kc <= a.cond_max);   // NaN and infinity fail the comparison
          km = fmaxf(km, kc);
        }
        if (bad) fl |= kStatusReslice | kStatusIllcond;
        guard = a.guard * fmaxf(1.f, km / a.cond_ref);
      }
    }
    c32 s;
    if (a.reg == 2) {
      c32 v = cscale(w, a.invC);
      s = c32{fminf(fmaxf(v.re, -a.box_r), a.box_r), fminf(fmaxf(v.im, -a.box_r), a.box_r)};
    } else {
      s = cscale(w, a.inv_den);
    }
    for (int t = 2; t <= a.T; ++t) {
      lam.re = fmaf(a.gamma, z.re - s.re, lam.re);
      lam.im = fmaf(a.gamma, z.im - s.im, lam.im);
      const c32 q = csub(s, lam);
      const c32 bq = bmat(q);
      z = c32{fmaf(a.rho, bq.re, yreg.re), fmaf(a.rho, bq.im, yreg.im)};
      w = (HALF == 0) ? consensus_w<G>(active ? cadd(z, lam) : cz(), buf, ls, u, g, a.C, a.Cp, sm, slot, nw)
                      : consensus<false>(active ? cadd(z, lam) : cz(), buf, ls, G, u, a.C, a.Cp, sm, slot, nw);
      buf ^= 1;
      if (a.reg == 2) {
        c32 v = cscale(w, a.invC);
        s = c32{fminf(fmaxf(v.re, -a.box_r), a.box_r), fminf(fmaxf(v.im, -a.box_r), a.box_r)};
      } else {
        s = cscale(w, a.inv_den);
      }
    }
    if (active && c == 0) {
      const size_t o = ((size_t)k * a.n_sym + n) * G + u;
      a.shat[o] = s;
      if (a.hard) {
        const int iI = slice_dim(s.re, a.kappa, a.L), iQ = slice_dim(s.im, a.kappa, a.L);
        a.hard[o] = (uint8_t)(iI + a.L * iQ);
        if (near_threshold(s.re, a.kappa, a.L, guard) || near_threshold(s.im, a.kappa, a.L, guard)) fl |= 2;
      }
      if (nonfinite(s)) fl |= 1;
    }
  }
  if (a.flags) {
    const int bits = group_flags<G>(fl, g);
    if (c == 0 && u == 0 && k < a.n_sc) {
      a.flags[k] = bits;
      if ((bits & kStatusReslice) && a.any) *a.any = a.epoch;
    }
  }
}

// Algorithm 2 over the symbols as columns.  A: the Grams as operands.  x, r and p
// are the same on every wave of the subcarrier; alpha and beta are scalars of a
// column pair.
template <int G>
__device__ __forceinline__ int syms_cg(const UlArgs& a, const c32 (&A)[G], int lane, int wave, float4* cons) {
  constexpr int P = 64 / G, NT = G / 16;
  const float sg = (lane & 8) ? 1.f : -1.f;   // [-xi | xr]
  const int wps = a.Cp / P, w0 = wave / wps * wps;
  const int k = a.blk * a.sc_per_block + wave / wps;
  int fl = 0, buf = 0;
  bool act[P];
#pragma unroll
  for (int p = 0; p < P; ++p) act[p] = k < a.n_sc && (wave - w0) * P + p < a.C;
  // sum of v . w over the users and the two parts of a symbol
  auto dot = [&](const f32x4 (&v)[NT], const f32x4 (&w)[NT]) {
    float d[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t)
      d[t] = fmaf(v[t][0], w[t][0], v[t][1] * w[t][1]) + fmaf(v[t][2], w[t][2], v[t][3] * w[t][3]);
    float e = d[0];
#pragma unroll
    for (int t = 1; t < NT; ++t) e += d[t];
    return pair_sum<32>(pair_sum<16>(e + swap_parts(e, 1.f)));
  };
  for (int n0 = 0; n0 < a.n_sym; n0 += 8) {
    f32x4 x[NT], r[NT], pv[NT];
    {
      f32x4 hy[P][NT];
      syms_hy<G, false>(a, n0, hy, lane, wave);
#pragma unroll
      for (int t = 0; t < NT; ++t) r[t] = x[t] = f32x4{};
#pragma unroll
      for (int p = 0; p < P; ++p) {
        if (act[p]) {
#pragma unroll
          for (int t = 0; t < NT; ++t) r[t] += hy[p][t];
        }
      }
    }
    syms_consensus<G>(r, cons, buf, lane, wave, wps);
#pragma unroll
    for (int t = 0; t < NT; ++t) pv[t] = r[t];
    float rr = dot(r, r);
    for (int it = 1; it <= a.T; ++it) {
      f32x4 e[NT];
#pragma unroll
      for (int t = 0; t < NT; ++t) e[t] = f32x4{};
#pragma unroll
      for (int p = 0; p < P; ++p) {
        if (act[p]) {
          f32x4 wc[NT];
          syms_matvec<G, false>(A, p, pv, wc, sg);
#pragma unroll
          for (int t = 0; t < NT; ++t) e[t] += wc[t];
        }
      }
      syms_consensus<G>(e, cons, buf, lane, wave, wps);
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) e[t][i] = fmaf(a.rho, pv[t][i], e[t][i]);
      const float pe = dot(pv, e);
      const float alpha = (rr > 0.f) ? rr * __builtin_amdgcn_rcpf(pe) : 0.f;
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          x[t][i] = fmaf(alpha, pv[t][i], x[t][i]);
          r[t][i] = fmaf(-alpha, e[t][i], r[t][i]);
        }
      const float rr_new = dot(r, r);
      const float beta = (rr > 0.f) ? rr_new * __builtin_amdgcn_rcpf(rr) : 0.f;
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) pv[t][i] = fmaf(beta, pv[t][i], r[t][i]);
      rr = rr_new;
    }
    if (wave == w0 && k < a.n_sc) fl |= syms_store<G>(a, x, k, n0, lane, a.guard);
  }
  return fl;
}

// ---------------------------------------------------------------------------
// Algorithm 2 (decentralized CG), FP32.  Each cluster keeps its own copy of
// x, r, p (the broadcast-w variant) and contributes w_c = H_c^H H_c p through
// its local Gram G_c held in registers (one matvec per iteration).
// ---------------------------------------------------------------------------
template <int G, bool SYMS = false>
__global__ void __launch_bounds__(512) dcg_ul_f32(UlArgs a) {
  a.blk = blockIdx.x;
  constexpr int P = 64 / G;
  extern __shared__ float4 smem_raw[];
  const int nw = blockDim.x >> 6;
  Smem sm = carve(reinterpret_cast<c32*>(smem_raw), nw);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave-uniform: addresses in SALU
  const int g = lane / G, u = lane % G;
  const int lp = wave * P + g;
  const int ls = lp / a.Cp, c = lp % a.Cp;
  const int k = a.blk * a.sc_per_block + ls;
  const bool active = (k < a.n_sc) && (c < a.C);
  const int slot = wave * 64 + lane;
  c32* line = sm.line + wave * 64;
  const int gbase = g * G;

  c32 A[G];
  // (the U = 16 Gram writes every entry of every lane's row: no clearing)
  if constexpr (G != 16) {
#pragma unroll
    for (int v = 0; v < G; ++v) A[v] = cz();
  }
  c32 hy0;
  if constexpr (G == 32)
    hy0 = gram_mfma_u32<false>(a, A, lane, wave, reinterpret_cast<float*>(line),
                               reinterpret_cast<float*>(sm.stage + wave * kStageWave));
  else if constexpr (G == 16)
    hy0 = gram_mfma_u16(a, A, lane, wave, sm.stage + wave * kStageWave);
  else if constexpr (G == 64)
    hy0 = gram_mfma_u64<0>(a, A, lane, wave, reinterpret_cast<float*>(line),
                               reinterpret_cast<float*>(sm.stage + wave * kStageWave));
  else
    hy0 = cluster_pass<G, true>(a.H, a.y, A, k, c, 0, u, g, lane, wave, active, a.B, a.S, G, a.n_sym, sm);

  if constexpr (SYMS) {
    rows_to_operands<G>(A);
    const int fl = syms_cg<G>(a, A, lane, wave, reinterpret_cast<float4*>(sm.stage));
    const int lead = wave * P;   // the wave's first problem
    syms_flags(a, fl, a.blk * a.sc_per_block + lead / a.Cp, lead % a.Cp == 0, lane);
    return;
  }

  int buf = 0;
  int fl = 0;   // status bits of this lane's outputs (bit 0 non-finite, bit 1 re-slice)
  for (int n = 0; n < a.n_sym; ++n) {
    c32 hy = hy0;
    if (n > 0) hy = cluster_pass<G, false>(a.H, a.y, A, k, c, n, u, g, lane, wave, active, a.B, a.S, G, a.n_sym, sm);
    // y^MRC = sum_c H_c^H y_c (consensus); r = p = y^MRC; x = 0
    c32 r = consensus_w<G>(active ? hy : cz(), buf, ls, u, g, a.C, a.Cp, sm, slot, nw);
    buf ^= 1;
    c32 pv = r, x = cz();
    float rr = group_sum<G>(r.re * r.re + r.im * r.im);
    for (int t = 1; t <= a.T; ++t) {
      const c32 wc = group_matvec<G>(A, pv, u, line, gbase);
      const c32 w = consensus_w<G>(active ? wc : cz(), buf, ls, u, g, a.C, a.Cp, sm, slot, nw);
      buf ^= 1;
      const c32 e = c32{fmaf(a.rho, pv.re, w.re), fmaf(a.rho, pv.im, w.im)};
      const float pe = group_sum<G>(pv.re * e.re + pv.im * e.im);
      // quotients by the hardware reciprocal (1 ulp) instead of a full division
      const float alpha = (rr > 0.f) ? rr * __builtin_amdgcn_rcpf(pe) : 0.f;
      x.re = fmaf(alpha, pv.re, x.re);
      x.im = fmaf(alpha, pv.im, x.im);
      r.re = fmaf(-alpha, e.re, r.re);
      r.im = fmaf(-alpha, e.im, r.im);
      const float rr_new = group_sum<G>(r.re * r.re + r.im * r.im);
      const float beta = (rr > 0.f) ? rr_new * __builtin_amdgcn_rcpf(rr) : 0.f;
      pv.re = fmaf(beta, pv.re, r.re);
      pv.im = fmaf(beta, pv.im, r.im);
      rr = rr_new;
    }
    if (active && c == 0) {
      const size_t o = ((size_t)k * a.n_sym + n) * G + u;
      a.shat[o] = x;
      if (a.hard) {
        const int iI = slice_dim(x.re, a.kappa, a.L), iQ = slice_dim(x.im, a.kappa, a.L);
        a.hard[o] = (uint8_t)(iI + a.L * iQ);
        if (near_threshold(x.re, a.kappa, a.L, a.guard) || near_threshold(x.im, a.kappa, a.L, a.guard)) fl |= 2;
      }
      if (nonfinite(x)) fl |= 1;
    }
  }
  if (a.flags) {
    const int bits = group_flags<G>(fl, g);
    if (c == 0 && u == 0 && k < a.n_sc) {
      a.flags[k] = bits;
      if ((bits & kStatusReslice) && a.any) *a.any = a.epoch;
    }
  }
}

// Inversions of one budgeted (P1) at most (see admm_dl_body; an FP32 model of the
// step over 6000 random problems, from a cold start each, needs two in 71 % of
// them, one in 24 % and four at most).
constexpr int kBudgetSteps = 12;

// ---------------------------------------------------------------------------
// Algorithm 3 (decentralized ADMM beamforming, epsilon = 0), S x S branch
// (S <= U), FP32.  Group size G = U.  The downlink cluster channel is
// H_c = (Hu_c)^T with Hu_c the S x U uplink block (reciprocity), read in place
// from the uplink layout.  Lane u holds column u of Hu_c (entries Hu_c[a][u],
// a < S) for m_c = H_c x_c; lane a < S holds row a of Hu_c for H_c^H v and
// row a of A_c^{-1}.
// ---------------------------------------------------------------------------
// BUDGET: every x-update is the budgeted step (P1) with ||x_c||^2 <= P_c.
// When the unconstrained step exceeds the budget, x = x(tau) = (H_c^H H_c +
// tau I)^{-1} H_c^H v with tau > 1/rho the root of ||x(tau)||^2 = P_c (the
// Lagrange multiplier of the budget is rho tau - 1).  The kernel keeps the
// inverse M at the shift tau_M of the symbol's last inversion (first 1/rho).  For a
// right-hand side r its powers u_j = M^{j+1} r, j = 0 .. 3, give x at any nearby
// shift, x(tau_M + d) = sum_j (-d)^j u_j, and through their inner products
// g_m = r^H M^{m+2} r the squared norm N(d) = sum_m (m + 1) (-d)^m g_m, m <= 6.
// d is the root of N(d) = P_c: a Halley step on 1/||x|| - 1/sqrt(P_c) (concave
// and increasing in tau, and nearly linear), polished on the polynomial where
// the series converges fast.  If the truncated tail of x is below FP32
// rounding the x-update is done, with no inversion at all; otherwise M is
// formed anew at tau_M + d and the step repeats.  The powers run in units of
// ||u_0|| and of the rate ||u_1|| / ||u_0||: g_6 falls with the eighth power of
// the shift and would leave FP32 at amplitudes of H of 1e3 or 1e-6.  The tail
// is estimated, not bounded: d^4 ||u_4|| with ||u_4|| taken as ||u_3||^2 / ||u_2||
// (at most 1.33 times too small in the 6000 problems of kBudgetSteps).
// The shift moves little from one x-update to the next, so a product (about 45
// instructions) replaces most inversions (about 900): B=256 U=32 C=16, 1200
// subcarriers, T=5, budgets binding on half of the clusters: 754 us with Newton's
// method and a Gram and an inversion per step (about 25 of them), 225 us in this
// form.  Relative error against FP64 at amplitudes of H of 1e-9 to 1e6 (rho fixed
// or scaled along), budgets of 1e-30 to 0.9 of the free energy and rho of 1e-12 to
// 1e12 on well-conditioned clusters: at most 8e-7, as at unit scale.
template <int G, int SG, bool BUDGET = false>
__device__ __forceinline__ void admm_dl_body(const DlArgs& a) {
  constexpr int P = 64 / G;
  extern __shared__ float4 smem_raw[];
  const int nw = blockDim.x >> 6;
  Smem sm = carve(reinterpret_cast<c32*>(smem_raw), nw);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave-uniform: addresses in SALU
  const int g = lane / G, u = lane % G;
  const int lp = wave * P + g;
  const int ls = lp / a.Cp, c = lp % a.Cp;
  const int k = blockIdx.x * a.sc_per_block + ls;
  const bool active = (k < a.n_sc) && (c < a.C);
  const int slot = wave * 64 + lane;
  c32* line = sm.line + wave * 64;
  const int gbase = g * G;
  const int S = a.S;
  // Entry (a, u) of the S x U uplink block Hu_c: row-major in the uplink
  // layout [n_sc][B][U] (strides U and 1), or read from the downlink layout
  // H^d [n_sc][U][B] (strides 1 and B).
  const bool dl_layout = a.h_layout == 1;
  const c32* Hk = a.H + (size_t)k * a.B * G + (dl_layout ? (size_t)c * S : (size_t)c * S * G);
  const size_t sa = dl_layout ? 1 : G, su = dl_layout ? (size_t)a.B : 1;

  // When SG = G / 2 the row of Hu_c that H_c^H v needs is split over two
  // lanes: lane u holds entries RS * (u / SG) .. + RS - 1 of row u % SG, and
  // the two half sums are combined by one exchange.  Otherwise lane u < S
  // holds the whole row u.
  constexpr bool SPLIT = (2 * SG == G);
  constexpr int RS = SPLIT ? SG : G;       // row entries held per lane
  const int ra = SPLIT ? (u % SG) : u;     // row of Hu_c held by this lane
  const int r0 = SPLIT ? RS * (u / SG) : 0;
  // With the matrix-core Gram (U = 32, S <= 16) the row copy hrow is formed
  // only after the inverse, from hcol through LDS, so that it is not live
  // during the Gram and the sweep (register budget of four waves per SIMD).
  constexpr bool LATE_H = (G == 32 && SG == 16);
  // There A_c and its inverse also take the split-row layout: lane u holds
  // entries 8 (u / 16) .. + 7 of row u % 16, so that all 32 lanes of the group
  // share the sweep and the products A_c^{-1} r.
  constexpr bool ASPLIT = LATE_H;
  constexpr int NR = ASPLIT ? 8 : SG;      // entries of A_c per lane
  // U = 64, S > 32: two copies of the 64 x 64 block beside A_c do not fit a lane's
  // registers (535 spilled, 1.5 KB of scratch per lane); H is read again for
  // every product instead, A_c is formed and inverted on the matrix cores.
  // B = 512, C = 8, S = 64, 1200 subcarriers, T = 5: 8.82 -> 1.29 ms; B = 92,
  // C = 2, S = 46, 1981 subcarriers: 3.01 -> 0.50 ms.
  constexpr bool STREAM = (G == 64 && SG == 64);
  constexpr int kUnroll = STREAM ? 4 : 16;   // (STREAM: 16 loads in flight)
  DlBlock64 hb{};
  if constexpr (STREAM) {
    const size_t ho = active ? (size_t)k * a.B * G + (dl_layout ? (size_t)c * S : (size_t)c * S * G) : 0;
    hb.rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<c32*>(a.H + ho), 0,
                                              active ? (dl_layout ? (63 * a.B + S) * 8 : S * 512) : 0, kBufferWord3);
    hb.S = S;
    hb.sa = dl_layout ? 8 : 512;
    hb.su = dl_layout ? a.B * 8 : 8;
  }
  c32 hcol[STREAM ? 1 : SG], hrow[STREAM ? 1 : RS], A[NR];
  if constexpr (!STREAM) {
#pragma unroll
    for (int i = 0; i < SG; ++i) hcol[i] = (active && i < S) ? Hk[(size_t)i * sa + (size_t)u * su] : cz();
  }
#pragma unroll
  for (int i = 0; i < NR; ++i) A[i] = cz();
  if constexpr (!LATE_H && !STREAM) {
#pragma unroll
    for (int i = 0; i < RS; ++i) hrow[i] = (active && ra < S) ? Hk[(size_t)ra * sa + (size_t)(r0 + i) * su] : cz();
  }
  // (H_c^H H_c)[a][b] = sum_u conj(Hu[a][u]) Hu[b][u] into M (rows a < S; M must
  // hold zeros), where it is not formed on the matrix cores.  Every lane of
  // the wave takes part.
  auto gram_into = [&](c32 (&M)[NR]) {
    // Row b of Hu_c is broadcast from the stage buffer of this wave.
    c32* stage = sm.stage + wave * kStageWave;
    for (int b = 0; b < S; ++b) {
      // lane u of the group publishes Hu[b][u] = hcol[b]
      c32 hb = cz();
#pragma unroll
      for (int i = 0; i < SG; ++i)
        if (i == b) hb = hcol[i];
      stage[lane] = hb;
      wave_lds_sync();
      c32 acc = cz();
#pragma unroll
      for (int v0 = 0; v0 < RS; v0 += 8) {
        c32 row[8];
        lds_read_vec<8>(stage + gbase + r0 + v0, row);
#pragma unroll
        for (int v = 0; v < 8; ++v) cmacc(acc, hrow[v0 + v], row[v]);
      }
      wave_lds_sync();
      if (SPLIT) acc = c32{pair_sum<SG>(acc.re), pair_sum<SG>(acc.im)};
#pragma unroll
      for (int i = 0; i < SG; ++i)
        if (i == b) M[i] = (u < S) ? acc : cz();
    }
  };
  // A_c = H_c^H H_c + rho^{-1} I_S (identity past S) and its inverse
  const float irho = 1.0f / a.rho;
  auto shift_invert = [&](c32 (&M)[NR], float tau) {
#pragma unroll
    for (int v = 0; v < NR; ++v)
      if (v == u) M[v].re += (u < S) ? tau : 1.0f;
    gj_invert<NR>(M, u, line, gbase);
  };
  // STREAM: Gram and inverse on the matrix cores (tau is the same on every lane)
  auto stream_invert = [&](c32 (&M)[NR], float tau) {
    if constexpr (STREAM) {
      UlArgs ua{};
      ua.H = a.H;
      ua.y = a.H;   // (not read)
      ua.n_sc = a.n_sc;
      ua.B = a.B;
      ua.C = a.C;
      ua.Cp = a.Cp;
      ua.S = 64;    // rows of H_c: the users
      ua.sc_per_block = a.sc_per_block;
      ua.rho = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(tau)));
      ua.blk = blockIdx.x;
      gram_mfma_u64<2, true>(ua, M, lane, wave, reinterpret_cast<float*>(line),
                             reinterpret_cast<float*>(sm.stage + wave * kStageWave), &hb);
    }
  };
  // the budgeted step inverts the Gram again at other shifts
  constexpr bool KEEP = BUDGET && ASPLIT;
  Tile16 gk[KEEP ? 2 : 1];
  if constexpr (ASPLIT) {
    Tile16 T[2];
    gram_dl_mfma_s16_u32(hcol, T, lane, g, u, sm.stage + wave * kStageWave);
    if constexpr (KEEP) {
      gk[0] = T[0];
      gk[KEEP ? 1 : 0] = T[1];
    }
    // (the vector sweep in both forms: a budget that never binds changes nothing)
    shift_invert_s16<false>(T, irho, irho, S, A, lane, line);
  } else if constexpr (STREAM) {
    stream_invert(A, irho);
  } else {
    gram_into(A);
    if constexpr (BUDGET) {
      shift_invert(A, irho);
    } else {
      // (in place: through the lambda the S > 16 forms kept part of A in scratch,
      // B = 232, U = 32, S = 29, 1681 subcarriers: 362 against 324 us)
#pragma unroll
      for (int v = 0; v < NR; ++v)
        if (v == u) A[v].re += (u < S) ? irho : 1.0f;
      gj_invert<NR>(A, u, line, gbase);
    }
  }
  if constexpr (LATE_H) {
    // Transpose the S x G tile of each problem through the wave's stage
    // buffer, one problem at a time: entry (i, w) at i (G + 2) + w.  The
    // pitch of G + 2 complex values keeps column pairs together and 16-byte
    // aligned, puts the rows that a read instruction touches into different
    // LDS banks, and makes every offset a compile-time constant
    // (SG (G + 2) = 544 values, the size of the stage buffer).
    c32* tile = sm.stage + wave * kStageWave;
    static_assert(SG * (G + 2) <= kStageWave, "tile exceeds the stage buffer");
    for (int pp = 0; pp < P; ++pp) {
      if (g == pp) {
#pragma unroll
        for (int i = 0; i < SG; ++i) tile[i * (G + 2) + u] = hcol[i];
      }
      wave_lds_sync();
      if (g == pp) {
#pragma unroll
        for (int m = 0; m < RS / 2; ++m) {
          const float4 v = *reinterpret_cast<const float4*>(tile + ra * (G + 2) + r0 + 2 * m);
          hrow[2 * m] = c32{v.x, v.y};
          hrow[2 * m + 1] = c32{v.z, v.w};
        }
      }
      wave_lds_sync();
    }
  }

  c32 Mt[BUDGET ? NR : 1];   // inverse at the shift tauM
  float tauM = irho;
  if constexpr (BUDGET) {
#pragma unroll
    for (int i = 0; i < NR; ++i) Mt[i] = A[i];
  }
  if constexpr (KEEP) {
    // the Gram waits in the wave's stage buffer, which is free from here on
    // with the split rows (lane-private slots)
    float* st = reinterpret_cast<float*>(sm.stage + wave * kStageWave) + lane;
#pragma unroll
    for (int i = 0; i < 16; ++i) st[64 * i] = (i & 4) ? gk[KEEP ? i >> 3 : 0].im[i & 3] : gk[KEEP ? i >> 3 : 0].re[i & 3];
  }

  // Broadcast line of the iterations, in the wave's stage buffer (free once
  // the Gram is formed): group g at g (G + 8), and with split rows the second
  // half of a group 4 entries further on, so that the (up to four) distinct
  // 16-byte addresses a read instruction touches fall into different LDS
  // banks.
  c32* bl = sm.stage + wave * kStageWave + g * (G + 8);
  const int bw = u + (SPLIT ? 4 * (u / RS) : 0);      // this lane's slot
  const int br = r0 + (SPLIT ? 4 * (r0 / RS) : 0);    // start of the half this lane reads
  int buf = 0;
  for (int n = 0; n < a.n_sym; ++n) {
    const size_t vo = ((size_t)k * a.n_sym + n);
    const c32 s = (k < a.n_sc) ? a.s[vo * G + u] : cz();
    c32 z = cscale(s, a.f0), lam = cz();
    if constexpr (BUDGET) {
      // Every symbol starts from 1/rho (with the shift kept from the symbol before,
      // its result would depend on that symbol).  The condition is for the
      // register allocator: without it U = 64, S = 17 .. 32 spills 247 registers
      // instead of 182 (C = 8, S = 24, 600 subcarriers: 1089 against 888 us), with
      // it S = 9 .. 16 spills 631 instead of 474 (2100 against 842 us).
      if (!(G == 64 && SG == 32) || n > 0) {
        tauM = irho;
#pragma unroll
        for (int i = 0; i < NR; ++i) Mt[i] = A[i];
      }
    }
    // H_c^H v: entry a held by lane a < S
    auto hhv = [&](c32 v) -> c32 {
      c32 acc = cz();
      if constexpr (ASPLIT) {
        // entry r0 + i of v sits in lane i of this lane's own 16-lane DPP row:
        // broadcast inside the FMAs, no LDS
        acc = matvec16c(hrow, v);
      } else {
        bl[bw] = v;
        wave_lds_sync();
#pragma unroll kUnroll
        for (int v0 = 0; v0 < RS; v0 += 4) {
          c32 vv[4];
          lds_read_vec<4>(bl + br + v0, vv);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            if constexpr (STREAM) cmacc(acc, hb.at(u, v0 + i), vv[i]);
            else cmacc(acc, hrow[v0 + i], vv[i]);
          }
        }
        wave_lds_sync();
      }
      if (SPLIT) acc = c32{pair_sum<SG>(acc.re), pair_sum<SG>(acc.im)};
      // the split-row product below takes entry a from both lanes of row a
      if constexpr (ASPLIT) return (ra < S) ? acc : cz();
      return (u < S) ? acc : cz();
    };
    // x_c = A_c^{-1} H_c^H (z + lambda), entry a held by lane a < S.  At
    // S = U (SG = G) the regularised Gram is as poorly conditioned as it gets
    // (condition numbers of a few hundred at S = U = 64), and the FP32 Gram
    // and Gauss-Jordan inverse lose about a factor three against an exactly
    // rounded solve there; one step of refinement whose residual is formed
    // from H itself, r - H_c^H (H_c x) - x / rho, wins it back.
    auto apply = [&](c32 v) -> c32 {
      const c32 r = hhv(v);
      // entry a of x_c on lane a < S (with the split rows, on both lanes of row a)
      c32 xa;
      if constexpr (ASPLIT)
        xa = matvec_split16(A, r);
      else
        xa = group_matvec<SG>(A, r, u, line, gbase);
      if constexpr (SG == G) {
        bl[bw] = xa;
        wave_lds_sync();
        c32 m = cz();
#pragma unroll kUnroll
        for (int v0 = 0; v0 < SG; v0 += 4) {
          c32 xv[4];
          lds_read_vec<4>(bl + v0, xv);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            if constexpr (STREAM) cmac(m, hb.at(v0 + i, u), xv[i]);
            else cmac(m, hcol[v0 + i], xv[i]);
          }
        }
        wave_lds_sync();
        const c32 q = hhv(m);
        const c32 res = (u < S) ? c32{fmaf(-irho, xa.re, r.re - q.re), fmaf(-irho, xa.im, r.im - q.im)} : cz();
        xa = cadd(xa, group_matvec<SG>(A, res, u, line, gbase));
      }
      if constexpr (BUDGET) {
        // padding cluster slots carry no budget
        const float Pc = active ? a.P[c] : 0.f;
        auto dot = [&](c32 p, c32 q) -> float {
          const float d = fmaf(p.re, q.re, p.im * q.im);
          if constexpr (ASPLIT) return group_sum<16>(d);   // both rows of 16 lanes hold every entry
          return group_sum<G>((u < S) ? d : 0.f);
        };
        auto mul = [&](c32 q) -> c32 {
          if constexpr (ASPLIT) return matvec_split16(Mt, q);
          else return group_matvec<SG>(Mt, q, u, line, gbase);
        };
        bool need = active && dot(xa, xa) > Pc;
        const float sp = sqrtf(Pc);
        if (need && sp == 0.f) {
          xa = cz();
          need = false;
        }
        for (int it = 0; __ballot(need); ++it) {   // wave-uniform: products and inversions are wave operations
          // u_j in units of 2^e0 and the shift in units of 2^-e1, so that every
          // g_m is of order one whatever the scales of H, rho and P_c: 2^e0 is
          // near ||M r||, 2^e1 near the rate ||M u_0|| / ||u_0|| (powers of two: exact)
          c32 u0 = mul(r);
          const int e0 = __builtin_amdgcn_frexp_expf(dot(u0, u0)) >> 1;
          u0 = cldexp(u0, -e0);
          c32 u1 = mul(u0);
          const float rate = dot(u0, u1);
          const int e1 = __builtin_amdgcn_frexp_expf(rate);
          u1 = cldexp(u1, -e1);
          const c32 u2 = cldexp(mul(u1), -e1), u3 = cldexp(mul(u2), -e1);
          const float g0 = dot(u0, u0), g1 = ldexpf(rate, -e1), g2 = dot(u1, u1), g3 = dot(u1, u2),
                      g4 = dot(u2, u2), g5 = dot(u2, u3), g6 = dot(u3, u3);
          const float sh = ldexpf(sp, -e0), dmin = ldexpf(irho - tauM, e1);
          // Halley's step, at most twice Newton's
          const float q = fminf(sqrtf(g0) / sh - 1.0f, 1e30f);
          float d = 2.f * q * g0 * g1 / fmaxf(g1 * g1, fmaf(3.f * q, fmaf(g1, g1, -g0 * g2), 2.f * g1 * g1));
          d = fmaxf(d, dmin);
          // rate of the series at its end (at most the largest eigenvalue of M; not
          // finite if u_3 overflows: then the step has to invert)
          const float lam = sqrtf(g6 / g4);
          bool conv = fabsf(d) * lam < 0.3f;
          if (conv) {
            // Newton on the polynomial N(d)
            float p = d;
#pragma unroll 1
            for (int j = 0; j < 3; ++j) {
              const float e = -p;
              const float N = fmaf(e, fmaf(e, fmaf(e, fmaf(e, fmaf(e, fmaf(e, 7.f * g6, 6.f * g5), 5.f * g4), 4.f * g3),
                                           3.f * g2), 2.f * g1), g0);
              const float D = fmaf(e, fmaf(e, fmaf(e, fmaf(e, fmaf(e, 42.f * g6, 30.f * g5), 20.f * g4), 12.f * g3),
                                           6.f * g2), 2.f * g1);   // -dN / dd
              p = fmaxf(fmaf(2.f * N, (sqrtf(N) / sh - 1.0f) / D, p), dmin);
            }
            conv = fabsf(p) * lam < 0.3f;   // (the root is where the polynomial holds)
            d = conv ? p : d;
          }
          const float d2 = d * d;
          // the tail of the series, about d^4 ||u_3|| lam, below half a unit of FP32 rounding
          const bool tail = conv && d2 * d2 * sqrtf(g6) * lam <= 3e-8f * sh;
          const bool done = tail || it >= kBudgetSteps;
          c32 xn = u0;   // (out of steps: the solution at the last shift)
          if (tail) {
            xn = c32{fmaf(-d, u1.re, u0.re), fmaf(-d, u1.im, u0.im)};
            xn = c32{fmaf(d2, fmaf(-d, u3.re, u2.re), xn.re), fmaf(d2, fmaf(-d, u3.im, u2.im), xn.im)};
          }
          const float e = dot(xn, xn);
          if (need && done) {
            // on the budget up to rounding; a final scale keeps it feasible
            xa = cldexp(cscale(xn, e > sh * sh ? sh / sqrtf(e) : 1.f), e0);
            need = false;
          }
          if (!__ballot(need)) break;
          // (a problem that is done or below its budget inverts at its old shift again)
          if (need) tauM += ldexpf(d, -e1);
          if constexpr (KEEP) {
            const float* st = reinterpret_cast<const float*>(sm.stage + wave * kStageWave) + lane;
            Tile16 T[2];
#pragma unroll
            for (int i = 0; i < 16; ++i) {
              if (i & 4) T[i >> 3].im[i & 3] = st[64 * i];
              else T[i >> 3].re[i & 3] = st[64 * i];
            }
            auto tau_of = [&](int l) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(tauM), l)); };
            shift_invert_s16<true>(T, tau_of(0), tau_of(32), S, Mt, lane, line);
          } else if constexpr (STREAM) {
            stream_invert(Mt, tauM);
          } else {
#pragma unroll
            for (int i = 0; i < NR; ++i) Mt[i] = cz();
            gram_into(Mt);
            shift_invert(Mt, tauM);
          }
        }
      }
      return xa;
    };
    c32 x = apply(z);
    for (int t = 2; t <= a.T; ++t) {
      // m_c = H_c x_c: m[u] = sum_a Hu[a][u] x[a]
      c32 m = cz();
      if constexpr (ASPLIT) {
        // x[a] sits in lane a of both 16-lane DPP rows of the group
        m = matvec16(hcol, x);
      } else {
        bl[bw] = x;
        wave_lds_sync();
#pragma unroll kUnroll
        for (int v0 = 0; v0 < SG; v0 += 4) {
          c32 xv[4];
          lds_read_vec<4>(bl + v0, xv);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            if constexpr (STREAM) cmac(m, hb.at(v0 + i, u), xv[i]);
            else cmac(m, hcol[v0 + i], xv[i]);
          }
        }
        wave_lds_sync();
      }
      const c32 wc = csub(m, lam);
      const c32 w = consensus_w<G>(active ? wc : cz(), buf, ls, u, g, a.C, a.Cp, sm, slot, nw);
      buf ^= 1;
      // Lemma 2: z_c = w_c + f (s - w) / C, f = max{0, 1 - eps / ||s - w||}
      // (f = 1 at eps = 0); every group holds the same s and w, one user per lane
      float fC = a.invC;
      if (a.eps > 0.f) {
        const float dre = s.re - w.re, dim = s.im - w.im;
        const float nd = sqrtf(group_sum<G>(dre * dre + dim * dim));
        fC = nd > a.eps ? a.invC * (1.0f - a.eps / nd) : 0.f;
      }
      z = c32{fmaf(fC, s.re - w.re, wc.re), fmaf(fC, s.im - w.im, wc.im)};
      lam.re = fmaf(-a.gamma, m.re - z.re, lam.re);
      lam.im = fmaf(-a.gamma, m.im - z.im, lam.im);
      x = apply(cadd(z, lam));
    }
    // optional common power scaling: beta = min(1, min_c sqrt(P_c / ||x_c||^2))
    // (with the budgeted step the budgets are met by every x-update instead)
    float beta = 1.0f;
    if (a.P && !BUDGET) {
      const float e = group_sum<G>((u < S) ? (x.re * x.re + x.im * x.im) : 0.f);
      float ratio = 1.0f;
      if (active && e > 0.f) ratio = fminf(1.0f, sqrtf(a.P[c] / e));
      c32* ab = sm.aux;
      if (u == 0) ab[wave * 64 + g] = c32{ratio, 0.f};
      __syncthreads();
      // problems of subcarrier ls occupy local problem indices ls*Cp .. ls*Cp+C-1
      for (int cc = 0; cc < a.C; ++cc) {
        const int q = ls * a.Cp + cc;
        beta = fminf(beta, ab[(q / P) * 64 + (q % P)].re);
      }
      __syncthreads();
    }
    if (active && u < S) a.x[vo * a.B + (size_t)c * S + u] = cscale(x, beta);
    if (active && c == 0 && u == 0 && a.beta) a.beta[vo] = beta;
  }
}

template <int G, int SG, bool BUDGET = false>
__global__ void __launch_bounds__(512) admm_dl_f32(DlArgs a) {
  admm_dl_body<G, SG, BUDGET>(a);
}

// The same with the register budget of four waves per SIMD: at B = 256,
// U = 32, C = 16 a subcarrier's workgroup has eight waves, and 128 VGPRs let
// two such workgroups share a CU instead of one.
template <int G, int SG>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4))) admm_dl_f32_w4(DlArgs a) {
  admm_dl_body<G, SG>(a);
}

// ---------------------------------------------------------------------------
// Packed FP16 channel: one 256-lane workgroup per (subcarrier, cluster) tile
// of S x U entries.  The tile's largest |component| m fixes the exponent
// e = floor(log2 m) - 14 (at least -126), so that the scaled entries H * 2^-e
// lie below 2^15 in magnitude (no overflow) and stay normal FP16 numbers (11
// significant bits) down to 2^-28 m; each entry is rounded to nearest even, and
// 2^e is stored as the tile's scale.  Tiles of up to 256 * kPackRegs entries
// stay in registers between the two steps (one read of H); larger tiles read
// the tile a second time.
// ---------------------------------------------------------------------------
constexpr int kPackRegs = 8;


__global__ void __launch_bounds__(256) pack_h16(const c32* __restrict__ H, uint32_t* __restrict__ H16,
                                                float* __restrict__ hscale, int B, int U, int C) {
  __shared__ float wmax[4];
  const int S = B / C;
  const int k = blockIdx.x / C, c = blockIdx.x % C;
  const size_t base = (size_t)k * B * U + (size_t)c * S * U;
  const int n = S * U;
  const bool cached = n <= 256 * kPackRegs;
  c32 r[kPackRegs];
  float m = 0.f;
  if (cached) {
#pragma unroll
    for (int j = 0; j < kPackRegs; ++j) {
      const int i = threadIdx.x + 256 * j;
      r[j] = i < n ? H[base + i] : cz();
      m = fmaxf(m, fmaxf(fabsf(r[j].re), fabsf(r[j].im)));
    }
  } else {
    for (int i = threadIdx.x; i < n; i += 256) {
      const c32 v = H[base + i];
      m = fmaxf(m, fmaxf(fabsf(v.re), fabsf(v.im)));
    }
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) m = fmaxf(m, __shfl_xor(m, d, 64));
  if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = m;
  __syncthreads();
  m = fmaxf(fmaxf(wmax[0], wmax[1]), fmaxf(wmax[2], wmax[3]));
  const int e = pack_exponent(m);
  if (cached) {
#pragma unroll
    for (int j = 0; j < kPackRegs; ++j) {
      const int i = threadIdx.x + 256 * j;
      if (i < n) H16[base + i] = pack_pair(r[j], e);
    }
  } else {
    for (int i = threadIdx.x; i < n; i += 256) H16[base + i] = pack_pair(H[base + i], e);
  }
  if (threadIdx.x == 0) hscale[blockIdx.x] = ldexpf(1.f, e);
}

// ---------------------------------------------------------------------------
// Per-subcarrier status: one 256-lane workgroup per subcarrier ORs "not
// finite" over the subcarrier's floats and writes the flag (every entry of
// the status array is written, so it needs no clearing).
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) scan_nonfinite(const float* __restrict__ x, size_t per_sc,
                                                      int32_t* __restrict__ status) {
  const float* p = x + (size_t)blockIdx.x * per_sc;
  int bad = 0;
  for (size_t i = threadIdx.x; i < per_sc; i += 256) bad |= !__builtin_isfinite(p[i]);
  bad = __syncthreads_or(bad);
  if (threadIdx.x == 0) status[blockIdx.x] = bad ? 1 : 0;
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
// A launch holds fewer than 2^32 work items (the runtime cuts a larger one off
// without an error): workgroups of `threads` per launch.
static long most_blocks(int threads) { return 0xffffffffu / (unsigned)threads; }

// The same call without its first k subcarriers.
template <int U>
static void skip(UlArgs& a, size_t k) {
  a.n_sc -= (int)k;
  if (a.H) a.H += k * a.B * U;
  a.y += k * a.n_sym * a.B;
  if (a.shat) a.shat += k * a.n_sym * U;
  if (a.hard) a.hard += k * a.n_sym * U;
  if (a.fac) a.fac += k * a.C * (U * (U + 1) / 2);
  if (a.H16) a.H16 += k * a.B * U;
  if (a.hscale) a.hscale += k * a.C;
  if (a.flags) a.flags += k;
}
template <int U>
static void skip(DlArgs& a, size_t k) {
  a.n_sc -= (int)k;
  a.H += k * a.B * U;
  a.s += k * a.n_sym * U;
  a.x += k * a.n_sym * a.B;
  if (a.beta) a.beta += k * a.n_sym;
}

template <int U, typename K, typename Args>
static hipError_t launch(K kernel, Args a, int nw, hipStream_t st) {
  for (;;) {
    const long blocks = ((long)a.n_sc + a.sc_per_block - 1) / a.sc_per_block, most = most_blocks(64 * nw);
    if (blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(kernel, dim3((unsigned)(blocks < most ? blocks : most)), dim3(64 * nw), smem_bytes(nw), st, a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || blocks <= most) return e;
    skip<U>(a, (size_t)most * a.sc_per_block);
  }
}

// Products of the block factors at U = 32 through LDS (see block_matvec_u32; the same
// bits either way): more than one wave per SIMD (256 CUs of four) and 16 products or
// more.
static bool line_products(long blocks, int nw, int n_sym, int T) {
  return (blocks + 255) / 256 * nw > 4 && (long)n_sym * T >= 16;
}

template <int G, int HALF, int INV>
static hipError_t launch_stage(const UlArgs& a, int nw, hipStream_t st, int stage) {
  if (stage == 1) return launch<G>(admm_ul_f32<G, HALF, INV, 1>, a, nw, st);
  if constexpr (INV == 0 && G >= 16) {
    if (symbol_columns(G, a.n_sym, a.B, a.S, a.C, a.T)) return launch<G>(admm_ul_f32<G, HALF, 0, 0, true>, a, nw, st);
  }
  if constexpr (G == 32 && HALF == 0) {
    if (line_products((a.n_sc + a.sc_per_block - 1) / a.sc_per_block, nw, a.n_sym, a.T))
      return launch<32>(admm_ul_f32<32, 0, 0, 0, false, true>, a, nw, st);
  }
  return launch<G>(admm_ul_f32<G, HALF, INV, 0>, a, nw, st);
}

hipError_t launch_factor_pack_u32(const UlArgs& a, int nw, hipStream_t st) {
  return launch<32>(admm_ul_f32<32, 0, 0, 4>, a, nw, st);
}

hipError_t launch_admm_ul_f32(const UlArgs& a, int U, int nw, hipStream_t st, int stage) {
  switch (U) {
    case 8: return launch_stage<8, 0, 0>(a, nw, st, stage);
    case 16: return launch_stage<16, 0, 0>(a, nw, st, stage);
    case 32: return launch_stage<32, 0, 0>(a, nw, st, stage);
    case 64: return launch_stage<64, 0, 0>(a, nw, st, stage);
  }
  return hipErrorInvalidValue;
}

template <int G, int HALF>
static hipError_t launch_mixed_inv(const UlArgs& a, int inv, int nw, hipStream_t st, int stage) {
  switch (inv) {
    case 0: return launch_stage<G, HALF, 0>(a, nw, st, stage);
    case 2: return launch_stage<G, HALF, 2>(a, nw, st, stage);
  }
  if constexpr (G == 32) {
    if (inv == 1) return launch_stage<G, HALF, 1>(a, nw, st, stage);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_admm_ul_mixed(const UlArgs& a, int U, int half, int inv, int nw, hipStream_t st, int stage) {
  if (U == 32)
    return half == 1 ? launch_mixed_inv<32, 1>(a, inv, nw, st, stage) : launch_mixed_inv<32, 2>(a, inv, nw, st, stage);
  if (U == 64)
    return half == 1 ? launch_mixed_inv<64, 1>(a, inv, nw, st, stage) : launch_mixed_inv<64, 2>(a, inv, nw, st, stage);
  return hipErrorInvalidValue;
}

hipError_t launch_admm_ul_f32_batch(const UlBatch& b, int U, int nw, int grid, hipStream_t st) {
  if (b.n < 1) return hipSuccess;
  bool syms = false, line = false;
  for (int i = 0; i < b.n; ++i) line = line || line_products(grid, nw, b.f[i].n_sym, b.f[i].T);
  for (int i = 0; i < b.n; ++i) syms = syms || symbol_columns(U, b.f[i].n_sym, b.f[i].B, b.f[i].S, b.f[i].C, b.f[i].T);
  // (24 frames of one large channel can exceed a launch)
  const int most = (int)most_blocks(64 * nw);
  const auto run = [&](auto kernel) {
    UlBatch part = b;
    for (int done = 0; done < grid; done += most) {
      const int g = grid - done < most ? grid - done : most;
      hipLaunchKernelGGL(kernel, dim3((unsigned)g), dim3((unsigned)(64 * nw)), smem_bytes(nw), st, part);
      for (int i = 0; i < b.n; ++i) part.first[i] -= most;
      if (grid - done <= most) break;
    }
  };
  switch (U) {
    case 8: run(admm_ul_f32_batch<8, false>); break;
    case 16: syms ? run(admm_ul_f32_batch<16, true>) : run(admm_ul_f32_batch<16, false>); break;
    case 32:
      syms   ? run(admm_ul_f32_batch<32, true, true>)
      : line ? run(admm_ul_f32_batch<32, false, true>)
             : run(admm_ul_f32_batch<32, false>);
      break;
    case 64: syms ? run(admm_ul_f32_batch<64, true>) : run(admm_ul_f32_batch<64, false>); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int U, int STAGE>
static hipError_t launch_resident(const UlArgs& a, int nw, hipStream_t st) {
  if (symbol_columns(U, a.n_sym, a.B, a.S, a.C)) return launch<U>(admm_ul_f32<U, 0, 0, STAGE, true>, a, nw, st);
  return launch<U>(admm_ul_f32<U, 0, 0, STAGE>, a, nw, st);
}

hipError_t launch_admm_ul_factored(const UlArgs& a, int U, int nw, hipStream_t st) {
  switch (U) {
    case 8: return launch<8>(admm_ul_f32<8, 0, 0, 2>, a, nw, st);
    case 16: return launch_resident<16, 2>(a, nw, st);
    case 32: return launch_resident<32, 2>(a, nw, st);
    case 64: return launch_resident<64, 2>(a, nw, st);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_admm_ul_factored_h16(const UlArgs& a, int U, int nw, hipStream_t st) {
  switch (U) {
    case 8: return launch<8>(admm_ul_f32<8, 0, 0, 3>, a, nw, st);
    case 16: return launch_resident<16, 3>(a, nw, st);
    case 32: return launch_resident<32, 3>(a, nw, st);
    case 64: return launch_resident<64, 3>(a, nw, st);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_pack_h16(const c32* H, uint32_t* H16, float* hscale, int n_sc, int B, int U, int C,
                           hipStream_t st) {
  const size_t tiles = (size_t)n_sc * C;
  if (tiles == 0) return hipSuccess;
  if (tiles > 0x7fffffff) return hipErrorInvalidValue;
  const size_t most = (size_t)most_blocks(256) / C;   // subcarriers per launch
  for (size_t k = 0; k < (size_t)n_sc; k += most) {
    const size_t n = (size_t)n_sc - k < most ? (size_t)n_sc - k : most;
    hipLaunchKernelGGL(pack_h16, dim3((unsigned)(n * C)), dim3(256), 0, st, H + k * B * U, H16 + k * B * U,
                       hscale + k * C, B, U, C);
  }
  return hipGetLastError();
}

hipError_t launch_scan_nonfinite(const float* x, size_t floats_per_sc, int n_sc, int32_t* status,
                                 hipStream_t st) {
  if (n_sc == 0) return hipSuccess;
  for (long k = 0; k < n_sc; k += most_blocks(256)) {
    const long n = n_sc - k < most_blocks(256) ? n_sc - k : most_blocks(256);
    hipLaunchKernelGGL(scan_nonfinite, dim3((unsigned)n), dim3(256), 0, st, x + k * floats_per_sc, floats_per_sc,
                       status + k);
  }
  return hipGetLastError();
}

template <int U>
static hipError_t launch_dcg(const UlArgs& a, int nw, hipStream_t st) {
  return symbol_columns(U, a.n_sym, a.B, a.S, a.C) ? launch<U>(dcg_ul_f32<U, true>, a, nw, st) : launch<U>(dcg_ul_f32<U>, a, nw, st);
}

hipError_t launch_dcg_ul_f32(const UlArgs& a, int U, int nw, hipStream_t st) {
  switch (U) {
    case 8: return launch<8>(dcg_ul_f32<8>, a, nw, st);
    case 16: return launch_dcg<16>(a, nw, st);
    case 32: return launch_dcg<32>(a, nw, st);
    case 64: return launch_dcg<64>(a, nw, st);
  }
  return hipErrorInvalidValue;
}

template <bool BUDGET>
static hipError_t launch_dl(const DlArgs& a, int U, int nw, hipStream_t st) {
  const int S = a.S;
  switch (U) {
    case 8: return launch<8>(admm_dl_f32<8, 8, BUDGET>, a, nw, st);
    case 16:
      return S <= 8 ? launch<16>(admm_dl_f32<16, 8, BUDGET>, a, nw, st) : launch<16>(admm_dl_f32<16, 16, BUDGET>, a, nw, st);
    case 32:
      if (S <= 8) return launch<32>(admm_dl_f32<32, 8, BUDGET>, a, nw, st);
      if (S <= 16) {
        // the budgeted form keeps a second inverse live (165 registers, three waves
        // per SIMD): capped at 128 an earlier build of it spilled 152 (240 -> 293 us
        // at B=256 C=16, 1200 subcarriers)
        if constexpr (BUDGET) return launch<32>(admm_dl_f32<32, 16, true>, a, nw, st);
        return launch<32>(admm_dl_f32_w4<32, 16>, a, nw, st);
      }
      return launch<32>(admm_dl_f32<32, 32, BUDGET>, a, nw, st);
    case 64:
      if (S <= 8) return launch<64>(admm_dl_f32<64, 8, BUDGET>, a, nw, st);
      if (S <= 16) return launch<64>(admm_dl_f32<64, 16, BUDGET>, a, nw, st);
      if (S <= 32) return launch<64>(admm_dl_f32<64, 32, BUDGET>, a, nw, st);
      return launch<64>(admm_dl_f32<64, 64, BUDGET>, a, nw, st);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_admm_dl_f32(const DlArgs& a, int U, int nw, hipStream_t st) {
  return (a.P && a.budget) ? launch_dl<true>(a, U, nw, st) : launch_dl<false>(a, U, nw, st);
}

}  // namespace dbp
