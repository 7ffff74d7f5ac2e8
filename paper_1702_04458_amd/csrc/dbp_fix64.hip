// Exact hard decisions: FP64 recomputation of the subcarriers whose FP32
// result lies near a decision threshold.
//
// The FP32 detection kernels flag every subcarrier with a soft value within a
// guard of a slicing threshold (Section III-A: nearest-point slicing of the
// equalized estimate; the guard is a stated multiple of the FP32 path's
// measured error).  For those subcarriers these kernels run the whole method
// again in FP64 -- Algorithm 1 (U x U branch: B_c = H_c^H H_c + rho I,
// y_c^reg, Lemma 1's consensus, the proximal steps E2-MMSE / E2-ZF / E2-BOX)
// or Algorithm 2 (decentralized CG, residual update with e^(t)) -- and
// overwrite the soft output (rounded to FP32) and the hard decision (taken in
// FP64).  The decisions then agree with an FP64 evaluation of the method
// everywhere except within about 1e-14 of a threshold.
//
// Work split: every workgroup scans the flags in windows (one chunk of 2,048
// subcarriers per wave), ranks the flagged subcarriers in index order and takes
// every G-th of them (G workgroups).  A few flagged subcarriers are
// the common case, so the pass is a latency problem: what counts is the serial
// chain of one subcarrier (Gram, U pivots, T products), not the chip's FP64
// rate.  A cluster's regularised Gram and inverse therefore stay in the
// registers of one team -- one wave for U <= 32, four waves for U = 64 -- in
// the accumulator layout of v_mfma_f64_16x16x4f64 (see team_gram), where four
// pivots need one published panel and no workgroup barrier for U <= 32, and an
// iteration one barrier (its consensus sum).
//   U <= 32: one workgroup per subcarrier, wave c is cluster c: one launch for
//     everything.
//   U = 64: the C inverses (64 KiB each) exceed a CU's registers, so a first
//     kernel with one workgroup per (subcarrier, cluster) inverts into the
//     workgroup's slot of the workspace and a second one iterates.  Every
//     entry of a slot is written before it is read, so the workspace needs no
//     clearing.
// Measured (profiler, time of the pass; before: tiles of 1024 threads exchanged
// through LDS with two barriers per pivot, inverses and products through the
// workspace, three launches at U >= 32):
//   B=128 U=16 C=8, 38,400 subcarriers, about 150 flagged      81 -> 25 us
//   eight frames of U=16 in one call                           48 -> 16 us
//   B=198 U=32 C=6, 731 subcarriers, 2 flagged                 73 -> 41 us
//   B=512 U=64 C=8, 1200 subcarriers, 14 flagged              250 -> 66 us
// What is left at U = 64: scan of the flags 5 us, Gram 11 us (256 FP64 MFMAs of
// 64 cycles per wave, and the first rows' latency), 16 block pivots 22 us, and
// the second kernel's reads of 512 KiB of inverses and 256 KiB of H.
#include <hip/hip_runtime.h>

#include "dbp_device.h"
#include "dbp_launch.h"

namespace dbp {
namespace {

constexpr int kFixThreads = 1024;

struct alignas(16) d2 {
  double re, im;
};

__device__ __forceinline__ d2 dzero() { return d2{0.0, 0.0}; }
__device__ __forceinline__ d2 dld(const c32* p) {
  const c32 v = *p;
  return d2{(double)v.re, (double)v.im};
}
// acc += conj(x) * y
__device__ __forceinline__ void dmacc(d2& acc, d2 x, d2 y) {
  acc.re = fma(x.re, y.re, acc.re);
  acc.re = fma(x.im, y.im, acc.re);
  acc.im = fma(x.re, y.im, acc.im);
  acc.im = fma(-x.im, y.re, acc.im);
}
// acc += x * y
__device__ __forceinline__ void dmac(d2& acc, d2 x, d2 y) {
  acc.re = fma(x.re, y.re, acc.re);
  acc.re = fma(-x.im, y.im, acc.re);
  acc.im = fma(x.re, y.im, acc.im);
  acc.im = fma(x.im, y.re, acc.im);
}

// i = clamp(floor((kappa x + L) / 2), 0, L - 1) in FP64, ties up
__device__ __forceinline__ int slice64(double x, double kappa, int L) {
  double i = floor((kappa * x + (double)L) / 2.0);
  i = fmin(fmax(i, 0.0), (double)(L - 1));
  return (int)i;
}

// True when the FP32 pass of this call flagged nothing (it stores the call's
// epoch at f.any when it flags a subcarrier): the pass then neither scans
// the flags nor recomputes anything.  A stale value from an earlier call
// differs from this call's epoch, so the test errs only towards scanning.
__device__ __forceinline__ bool nothing_flagged(const FixArgs& f) { return f.any && *f.any != f.epoch; }

// The frames of one launch: a single call's arguments or a batch's.
struct OneFrame {
  const FixArgs& f;
  __device__ __forceinline__ int n() const { return 1; }
  __device__ __forceinline__ const FixArgs& at(int) const { return f; }
};
struct ManyFrames {
  const FixBatch& b;
  __device__ __forceinline__ int n() const { return b.n; }
  __device__ __forceinline__ const FixArgs& at(int i) const { return b.f[i]; }
};

// Bit i set: frame i has flagged subcarriers (at most 24 frames; lane i of
// every wave looks at frame i, so the loads are in flight together).
__device__ __forceinline__ unsigned flagged_frames(const OneFrame& fr) { return nothing_flagged(fr.f) ? 0u : 1u; }
__device__ __forceinline__ unsigned flagged_frames(const ManyFrames& fr) {
  const int lane = threadIdx.x & 63;
  const bool on = lane < fr.n() && !nothing_flagged(fr.at(lane < fr.n() ? lane : 0));
  return (unsigned)__ballot(on);
}

// Flags per wave in one scan of the flag array (kScan coalesced loads in
// flight), and the capacity of a workgroup's list.
constexpr int kScan = 32;
constexpr int kChunk = 64 * kScan;
constexpr int kListCap = kChunk;

// One workgroup's share of a window: (frame, subcarrier) pairs.
struct FixList {
  int k[kListCap];
  unsigned char fr[kListCap];
  int wsum[kFixThreads / 64];
};

// The subcarriers of all flagged frames (mask act) form one sequence of chunks
// of kChunk, a frame's chunks in order and its last one partly filled.  A
// window is `wt` chunks from chunk0 on, one per wave (wt is at most the waves
// of the workgroup).  Every workgroup ranks the flagged subcarriers of the
// window in index order and takes those of rank q0, q0 + G, ... into
// list[0 .. n), which must fit kListCap, with (G, q0) = share(number of flagged
// subcarriers of the window); returns n, and that number in *total.
struct Share {
  int G, q0;
};
// (wt so that a workgroup's share, at most wt kChunk / G, fits the list)
__device__ __forceinline__ int fix_window(int waves, int G) { return waves < G ? waves : G; }
__device__ __forceinline__ long frame_chunks(const FixArgs& f) { return ((long)f.n_sc + kChunk - 1) / kChunk; }
template <class FR>
__device__ __forceinline__ long fix_chunks(const FR& fr, unsigned act) {
  long c = 0;
  for (int i = 0; i < fr.n(); ++i)
    if ((act >> i) & 1u) c += frame_chunks(fr.at(i));
  return c;
}

template <class FR, class F>
__device__ __forceinline__ int collect_window(const FR& fr, unsigned act, long chunk0, int wt, FixList& L, int* total_out,
                                              F share) {
  __syncthreads();   // the previous round's list and sums are no longer read
  const int lane = threadIdx.x & 63, nwv = blockDim.x >> 6;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // this wave's chunk (wave-uniform)
  const int32_t* flags = nullptr;
  long base = 0, end = 0;
  int frame = 0;
  long ch = chunk0 + wv;
  for (int i = 0; i < fr.n() && wv < wt; ++i) {
    if (!((act >> i) & 1u)) continue;
    const long nc = frame_chunks(fr.at(i));
    if (ch >= 0 && ch < nc) {
      flags = fr.at(i).flags;
      end = fr.at(i).n_sc;
      base = ch * kChunk;
      frame = i;
    }
    ch -= nc;
  }
  unsigned bits = 0;   // bit i: flag base + 64 i + lane
  int mine = 0;        // flagged subcarriers of the chunk
  if (flags) {
    // (no branches and no masks kept per flag: a lane past the end reads the last
    // flag again and drops it from its bits)
    const int room = (int)(end - base < kChunk ? end - base : kChunk);   // >= 1
    int l = lane;
    asm volatile("" : "+v"(l));   // (or the 32 offsets are kept over the windows)
    int v[kScan];
#pragma unroll
    for (int i = 0; i < kScan; ++i) {
      const int k = 64 * i + l;
      v[i] = flags[base + (k < room ? k : room - 1)];
    }
#pragma unroll
    for (int i = 0; i < kScan; ++i) bits |= (v[i] & kStatusReslice) ? 1u << i : 0u;
    const int left = room - lane;          // this lane's flags are those of 64 i < left
    const int valid = left > 0 ? (left + 63) / 64 : 0;
    bits &= valid >= kScan ? ~0u : (1u << valid) - 1u;
    const int own = __popc(bits);          // 0 .. 32
#pragma unroll
    for (int p = 0; p < 6; ++p) mine += __popcll(__ballot((own >> p) & 1)) << p;
  }
  if (lane == 0) L.wsum[wv] = mine;
  __syncthreads();
  int q = 0, total = 0;   // q: rank of the chunk's first flagged subcarrier
  for (int w = 0; w < nwv; ++w) {
    const int c = L.wsum[w];
    q += w < wv ? c : 0;
    total += c;
  }
  const Share sh = share(total);
  const int G = sh.G, q0 = sh.q0;
  if (mine > 0) {   // wave-uniform
    // (rolled: 32 copies with their divisions are 10 KB of code, fetched anew by
    // every launch)
#pragma unroll 1
    for (int i = 0; i < kScan; ++i) {
      const bool on = (bits >> i) & 1u;
      const unsigned long long m = __ballot(on);
      if (!m) continue;   // uniform
      const int r = q + __popcll(m & ((1ull << lane) - 1)) - q0;
      if (on && r >= 0 && r % G == 0) {
        L.k[r / G] = (int)(base + 64 * i + lane);
        L.fr[r / G] = (unsigned char)frame;
      }
      q += __popcll(m);
    }
  }
  __syncthreads();
  *total_out = total;
  return total > q0 ? (total - q0 + G - 1) / G : 0;
}

// Calls body(frame, subcarrier) for workgroup g's share of all flagged
// subcarriers: those of rank g, g + G, ... over all windows, from rank `from` on.
template <class FR, class Body>
__device__ __forceinline__ void for_flagged(const FR& fr, unsigned act, int G, int g, long from, FixList& L, Body body) {
  const int wt = fix_window(blockDim.x >> 6, G);
  const long chunks = fix_chunks(fr, act);
  long seen = 0;
  for (long c0 = 0; c0 < chunks; c0 += wt) {
    const int q0 = (int)(((long)g - seen % G + G) % G);
    int total = 0;
    const int nl = collect_window(fr, act, c0, wt, L, &total, [&](int) { return Share{G, q0}; });
    for (int q = 0; q < nl; ++q)
      if (seen + q0 + (long)q * G >= from)
        body(fr.at(__builtin_amdgcn_readfirstlane((int)L.fr[q])), __builtin_amdgcn_readfirstlane(L.k[q]));
    seen += total;
  }
}

// Proximal step of Lemma 1 on the summed vector w (E2-MMSE / E2-ZF: w / den,
// den = N0 / (rho Es) + C; E2-BOX: clip of w / C to the QAM box).  f.inv_den
// holds the denominator itself (FP64 divides by it).
__device__ __forceinline__ d2 prox64(const FixArgs& f, d2 w) {
  if (f.reg == 2) {
    const double vr = w.re * f.invC, vi = w.im * f.invC;
    return d2{fmin(fmax(vr, -f.box_r), f.box_r), fmin(fmax(vi, -f.box_r), f.box_r)};
  }
  return d2{w.re / f.inv_den, w.im / f.inv_den};
}

__device__ __forceinline__ void write_out(const FixArgs& f, int k, int n, int u, d2 s) {
  const size_t o = ((size_t)k * f.n_sym + n) * f.U + u;
  f.shat[o] = c32{(float)s.re, (float)s.im};
  if (f.hard) f.hard[o] = (uint8_t)(slice64(s.re, f.kappa, f.L) + f.L * slice64(s.im, f.kappa, f.L));
}

// ---------------------------------------------------------------------------
// One cluster's U x U matrix in the registers of a team.  Lane l = 16 ti + tj
// holds the entries of rows 4 a + ti (a < NA; plus 16 tw for wave tw of a U = 64
// team) and columns 16 b + tj (b < NB): the accumulator layout of
// v_mfma_f64_16x16x4f64 (register r of a tile: row 4 r + l / 16, column l % 16).
// U = 8 uses the U = 16 layout with rows and columns 8 .. 15 zero (their
// diagonal rho keeps them decoupled).
// ---------------------------------------------------------------------------
typedef double f64x4 __attribute__((ext_vector_type(4)));

template <int U>
struct Team {
  static constexpr int TW = U == 64 ? 4 : 1;    // waves
  static constexpr int N = U < 16 ? 16 : U;     // padded matrix side
  static constexpr int NA = U == 32 ? 8 : 4;    // rows per lane
  static constexpr int NB = N / 16;             // columns per lane
  static constexpr int NI = NA / 4;             // 16-row tiles per wave
  // LDS of a team: panels of four rows and their 4 x 4 pivot block (two in turn
  // when the team has several waves; the accesses of one wave are in order)
  static constexpr int kPanel = 4 * N + 16;       // in d2
  static constexpr int kLds = (TW > 1 ? 2 : 1) * kPanel;
};

// This wave's 16 x 16 tiles: row tile i, column tile b (for U = 64 its one row
// tile is tw).
template <int U>
struct Tiles {
  f64x4 re[Team<U>::NI][Team<U>::NB], im[Team<U>::NI][Team<U>::NB];
};

template <int U>
__device__ __forceinline__ void team_sync() {
  if constexpr (Team<U>::TW > 1) __syncthreads();
  else wave_lds_sync();
}

// B_c = H_c^H H_c + rho I on the FP64 matrix cores (K runs over four antenna
// rows: lane l supplies H[s0 + l / 16][16 b + l % 16]), and entries 16 b + tj
// of H_c^H y_c when HY (the same for every ti).  The loads of the next 4 D rows
// are in flight while the current ones are multiplied.
template <int U, bool HY, int D = 4>
__device__ __forceinline__ void team_gram(const c32* __restrict__ Hc, const c32* __restrict__ yc, int S, double rho,
                                          int tw, int lane, Tiles<U>& M, d2 (&hy)[Team<U>::NB]) {
  constexpr int NB = Team<U>::NB, NI = Team<U>::NI;
  const int ti = lane >> 4, tj = lane & 15;
  auto& re = M.re;
  auto& im = M.im;
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int b = 0; b < NB; ++b) re[i][b] = im[i][b] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int b = 0; b < NB; ++b) hy[b] = dzero();
  constexpr int NC = U == 64 ? NB + 1 : NB;   // U = 64: entry NB is the A operand, column block tw
  c32 cur[D][NC], nxt[D][NC], ycur[D], ynxt[D];
  auto fetch = [&](int s0, c32 (&h)[D][NC], c32 (&yv)[D]) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      const int s = s0 + 4 * d + ti;
      const bool ok = s < S && (U >= 16 || tj < U);   // rows past S and padding columns add nothing
#pragma unroll
      for (int b = 0; b < NC; ++b) h[d][b] = ok ? Hc[(size_t)s * U + 16 * (b < NB ? b : tw) + tj] : c32{0.f, 0.f};
      if constexpr (HY) yv[d] = s < S ? yc[s] : c32{0.f, 0.f};
    }
  };
  fetch(0, cur, ycur);
  for (int s0 = 0; s0 < S; s0 += 4 * D) {
    if (s0 + 4 * D < S) fetch(s0 + 4 * D, nxt, ynxt);
#pragma unroll
    for (int d = 0; d < D; ++d) {
      if (s0 + 4 * d >= S) break;   // uniform
      d2 h[NC];
#pragma unroll
      for (int b = 0; b < NC; ++b) {
        h[b] = d2{(double)cur[d][b].re, (double)cur[d][b].im};
        if constexpr (HY) dmacc(hy[b], h[b], d2{(double)ycur[d].re, (double)ycur[d].im});
      }
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const d2 ha = h[U == 64 ? NB : i];   // the A operand: the columns that become this tile's rows
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          re[i][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(ha.re, h[b].re, re[i][b], 0, 0, 0);
          im[i][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(ha.re, h[b].im, im[i][b], 0, 0, 0);
        }
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          re[i][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(ha.im, h[b].im, re[i][b], 0, 0, 0);
          im[i][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(-ha.im, h[b].re, im[i][b], 0, 0, 0);
        }
      }
    }
#pragma unroll
    for (int d = 0; d < D; ++d) {
#pragma unroll
      for (int b = 0; b < NC; ++b) cur[d][b] = nxt[d][b];
      ycur[d] = ynxt[d];
    }
  }
  const int r0 = U == 64 ? 16 * tw : 0;
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int b = 0; b < NB; ++b)
        if (r0 + 16 * i + 4 * r + ti == 16 * b + tj) re[i][b][r] += rho;
}

// Sums over ti of x on even and of y on odd rows of 16 lanes (D = 16: lanes l
// and l ^ 16), or of x in the lower and of y in the upper wave half (D = 32).
template <int D>
__device__ __forceinline__ double swap_add(double x, double y) {
  const uint64_t u = __builtin_bit_cast(uint64_t, x), v = __builtin_bit_cast(uint64_t, y);
  auto swap = [](unsigned a, unsigned b) {
    if constexpr (D == 16) return __builtin_amdgcn_permlane16_swap(a, b, false, false);
    else return __builtin_amdgcn_permlane32_swap(a, b, false, false);
  };
  const auto lo = swap((unsigned)u, (unsigned)v), hi = swap((unsigned)(u >> 32), (unsigned)(v >> 32));
  return __builtin_bit_cast(double, (uint64_t)lo[0] | ((uint64_t)hi[0] << 32)) +
         __builtin_bit_cast(double, (uint64_t)lo[1] | ((uint64_t)hi[1] << 32));
}
// Sum over ti of v[b], handed to the lanes with b = ti mod NB: a wave's vectors
// have entry l % N on lane l.
template <int NB>
__device__ __forceinline__ double ti_sum(double a, double b, double c, double d) {
  if constexpr (NB == 4) return swap_add<32>(swap_add<16>(a, b), swap_add<16>(c, d));
  const double s = swap_add<16>(a, NB == 2 ? b : a);
  return swap_add<32>(s, s);
}
template <int NB>
__device__ __forceinline__ d2 ti_sum(const d2 (&v)[NB]) {
  constexpr int b = NB > 1 ? 1 : 0, c = NB > 2 ? 2 : 0, d = NB > 2 ? 3 : 0;
  return d2{ti_sum<NB>(v[0].re, v[b].re, v[c].re, v[d].re), ti_sum<NB>(v[0].im, v[b].im, v[c].im, v[d].im)};
}

// 1 / d: the hardware estimate and two Newton steps
__device__ __forceinline__ double rcp64(double d) {
  double p = __builtin_amdgcn_rcp(d);
  p = fma(fma(-d, p, 1.0), p, p);
  return fma(fma(-d, p, 1.0), p, p);
}

// In-place inverse of the team's Hermitian positive definite matrix: block
// Gauss-Jordan elimination, four pivots per step.  Rows 4 k .. 4 k + 3 are one
// accumulator register of the lanes of one row tile (row group ti holds row
// 4 k + ti), so a step publishes that panel W (4 x N) with its 4 x 4 pivot block
// P, and the update of every 16 x 16 tile is one K = 4 complex product on the
// matrix cores.  With the pivot columns of W replaced by the identity, and the
// pivot rows and columns of the matrix by zeros, the whole sweep
//   S_ij -= S_iP P^{-1} W_j,  S_Pj = P^{-1} W_j,  S_iP = -S_iP P^{-1},  S_PP = P^{-1}
// is S += A W with A_i = -S_iP P^{-1} (rows of P^{-1} for i in P).  Row P gives
// column P: S_iP is conj(W_i), negated for rows i already swept, hence A_i =
// -+conj(V_i) with V = P^{-1} W, and lane (ti, tj) needs the one entry
// V[ti][16 I + tj] for row tile I.  P^{-1} is applied through its 2 x 2 blocks
// (two reciprocals on the chain instead of four).
// Against one pivot per step (one published row, vector FMAs on the tiles) the
// chain is what counts: U = 64 has 16 barriers instead of 64.
template <int U>
__device__ __forceinline__ void team_invert(Tiles<U>& M, int tw, int lane, d2* lds) {
  constexpr int N = Team<U>::N, NB = Team<U>::NB, NI = Team<U>::NI, TW = Team<U>::TW;
  const int ti = lane >> 4, tj = lane & 15;
#pragma unroll 1
  for (int k4 = 0; k4 < N / 4; ++k4) {
    d2* W = lds + (TW > 1 ? (k4 & 1) * Team<U>::kPanel : 0);   // [4][N]
    d2* Pb = W + 4 * N;                                        // [4][4]
    const int Ik = k4 >> 2, r = k4 & 3;                        // the panel's row tile and register (uniform)
    const bool mine = (tj >> 2) == r;                          // this lane's column of tile Ik is a pivot column
    // publish register R of row tile I, and clear it
    auto publish = [&](auto Ic, auto Rc) {
      constexpr int I = decltype(Ic)::value, R = decltype(Rc)::value;
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        const d2 v = d2{M.re[I][b][R], M.im[I][b][R]};
        const bool piv = b == Ik && mine;
        if (piv) Pb[4 * ti + (tj & 3)] = v;
        W[ti * N + 16 * b + tj] = piv ? d2{ti == (tj & 3) ? 1.0 : 0.0, 0.0} : v;
        M.re[I][b][R] = 0.0;
        M.im[I][b][R] = 0.0;
      }
    };
    auto publish_tile = [&](auto Ic) {
      if (r == 0) publish(Ic, std::integral_constant<int, 0>{});
      else if (r == 1) publish(Ic, std::integral_constant<int, 1>{});
      else if (r == 2) publish(Ic, std::integral_constant<int, 2>{});
      else publish(Ic, std::integral_constant<int, 3>{});
    };
    if constexpr (TW > 1) {
      if (tw == Ik) publish_tile(std::integral_constant<int, 0>{});
    } else if (NI == 1 || Ik == 0) {
      publish_tile(std::integral_constant<int, 0>{});
    } else {
      publish_tile(std::integral_constant<int, NI - 1>{});
    }
    // clear the pivot columns (column tile Ik)
#pragma unroll
    for (int b = 0; b < NB; ++b)
      if (b == Ik) {   // uniform
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            M.re[i][b][q] = mine ? 0.0 : M.re[i][b][q];
            M.im[i][b][q] = mine ? 0.0 : M.im[i][b][q];
          }
      }
    team_sync<U>();
    // operands: the pivot block's upper triangle, the panel's columns that are
    // this wave's rows, and this lane's panel row
    d2 w[NI][4], Bv[NB];
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) w[i][q] = W[q * N + 16 * (TW > 1 ? tw : i) + tj];
    const double p00 = Pb[0].re, p11 = Pb[5].re, p22 = Pb[10].re, p33 = Pb[15].re;
    const d2 p01 = Pb[1], p02 = Pb[2], p03 = Pb[3], p12 = Pb[6], p13 = Pb[7], p23 = Pb[11];
#pragma unroll
    for (int b = 0; b < NB; ++b) Bv[b] = W[ti * N + 16 * b + tj];
    auto conjd = [](d2 x) { return d2{x.re, -x.im}; };
    // X = P_11^{-1} P_12 and the inverse of the Schur complement
    const double i1 = rcp64(fma(p00, p11, -fma(p01.re, p01.re, p01.im * p01.im)));
    const double a00 = p11 * i1, a11 = p00 * i1;
    const d2 a01 = d2{-p01.re * i1, -p01.im * i1}, a10 = conjd(a01);
    auto mul_a = [&](d2 x0, d2 x1, d2& t0, d2& t1) {   // t = P_11^{-1} x
      t0 = d2{a00 * x0.re, a00 * x0.im};
      dmac(t0, a01, x1);
      t1 = d2{a11 * x1.re, a11 * x1.im};
      dmac(t1, a10, x0);
    };
    d2 x02, x12, x03, x13;
    mul_a(p02, p12, x02, x12);
    mul_a(p03, p13, x03, x13);
    auto sub_h = [](d2 acc, d2 y0, d2 z0, d2 y1, d2 z1) {   // acc - conj(y0) z0 - conj(y1) z1
      dmacc(acc, d2{-y0.re, -y0.im}, z0);
      dmacc(acc, d2{-y1.re, -y1.im}, z1);
      return acc;
    };
    const double s22 = sub_h(d2{p22, 0.0}, p02, x02, p12, x12).re, s33 = sub_h(d2{p33, 0.0}, p03, x03, p13, x13).re;
    const d2 s23 = sub_h(p23, p02, x03, p12, x13);
    const double i2 = rcp64(fma(s22, s33, -fma(s23.re, s23.re, s23.im * s23.im)));
    const double c22 = s33 * i2, c33 = s22 * i2;
    const d2 c23 = d2{-s23.re * i2, -s23.im * i2}, c32_ = conjd(c23);
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      d2 t0, t1;
      mul_a(w[i][0], w[i][1], t0, t1);
      const d2 r2 = sub_h(w[i][2], p02, t0, p12, t1), r3 = sub_h(w[i][3], p03, t0, p13, t1);
      d2 v2 = d2{c22 * r2.re, c22 * r2.im}, v3 = d2{c33 * r3.re, c33 * r3.im};
      dmac(v2, c23, r3);
      dmac(v3, c32_, r2);
      const d2 n2 = d2{-v2.re, -v2.im}, n3 = d2{-v3.re, -v3.im};
      dmac(t0, x02, n2);
      dmac(t0, x03, n3);
      dmac(t1, x12, n2);
      dmac(t1, x13, n3);
      const d2 v = ti < 2 ? (ti == 0 ? t0 : t1) : (ti == 2 ? v2 : v3);
      // -+conj(v): rows already swept and the pivot rows take the plus sign
      const bool swept = 16 * (TW > 1 ? tw : i) + tj < 4 * (k4 + 1);
      const double ar = swept ? v.re : -v.re, ai = swept ? -v.im : v.im;
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        M.re[i][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(ar, Bv[b].re, M.re[i][b], 0, 0, 0);
        M.im[i][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(ar, Bv[b].im, M.im[i][b], 0, 0, 0);
      }
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        M.re[i][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(-ai, Bv[b].im, M.re[i][b], 0, 0, 0);
        M.im[i][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(ai, Bv[b].re, M.im[i][b], 0, 0, 0);
      }
    }
  }
  team_sync<U>();   // the panels may be overwritten
}

// This lane's part (rows s = ti mod 4) of entries 16 b + tj of H_c^H y_c.
template <int U>
__device__ __forceinline__ void team_hy(const c32* __restrict__ Hc, const c32* __restrict__ yc, int S, int lane,
                                        d2 (&hy)[Team<U>::NB]) {
  constexpr int NB = Team<U>::NB;
  const int ti = lane >> 4, tj = lane & 15;
#pragma unroll
  for (int b = 0; b < NB; ++b) hy[b] = dzero();
#pragma unroll 4
  for (int s = ti; s < S; s += 4) {
    const d2 yv = dld(yc + s);
#pragma unroll
    for (int b = 0; b < NB; ++b)
      if (U >= 16 || tj < U) dmacc(hy[b], dld(Hc + (size_t)s * U + 16 * b + tj), yv);
  }
}

// Inverses of a wave's cluster for the iterations: in registers (U <= 32).
template <int U>
struct RegInverse {
  Tiles<U> M;
  // acc[b] += sum over the lane's rows i of conj(M[i][16 b + tj]) line[i]
  __device__ __forceinline__ void apply(d2 (&acc)[Team<U>::NB], const d2* line, int lane) const {
    const int ti = lane >> 4;
#pragma unroll
    for (int a = 0; a < Team<U>::NA; ++a) {
      const d2 qi = line[4 * a + ti];
#pragma unroll
      for (int b = 0; b < Team<U>::NB; ++b) dmacc(acc[b], d2{M.re[a / 4][b][a % 4], M.im[a / 4][b][a % 4]}, qi);
    }
  }
};

// U = 64: a cluster's 64 x 64 block in the order [16-row block][a][b][lane] of
// the team layout (coalesced both ways).  kHeld of the four 16-row blocks stay
// in registers over all products, the rest is read again from the L2.
constexpr int kBlk64 = 16 * 64;   // complex values of one 16-row block
constexpr int kHeld = 2;
struct SlotInverse {
  d2 held[kHeld][4][4];
  const d2* Mc;
  __device__ __forceinline__ void load(const d2* m, int lane) {
    Mc = m + lane;
#pragma unroll
    for (int i = 0; i < kHeld * 16; ++i) held[i / 16][i / 4 % 4][i % 4] = Mc[i * 64];
  }
  __device__ __forceinline__ void apply(d2 (&acc)[4], const d2* line, int lane) const {
    const int ti = lane >> 4;
    // (eight loads in flight per step)
#pragma unroll 1
    for (int a = 4 * kHeld; a < 16; a += 2) {
      d2 m[2][4];
#pragma unroll
      for (int j = 0; j < 8; ++j) m[j / 4][j % 4] = Mc[(4 * a + j) * 64];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const d2 qi = line[4 * (a + j) + ti];
#pragma unroll
        for (int b = 0; b < 4; ++b) dmacc(acc[b], m[j][b], qi);
      }
    }
#pragma unroll
    for (int I = 0; I < kHeld; ++I)
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        const d2 qi = line[16 * I + 4 * a + ti];
#pragma unroll
        for (int b = 0; b < 4; ++b) dmacc(acc[b], held[I][a][b], qi);
      }
  }
};

// LDS (in d2) of a workgroup of nw waves: per wave a line for the products'
// operands (U <= 32: inside the team's panel, which is free by then), and two
// consensus buffers of nw rows.  (U = 64: larger than the panels of two teams,
// which use the same space before the iterations.)
template <int U>
constexpr int kLineStride = U == 64 ? 64 : Team<U>::kLds;
template <int U>
constexpr int fix_lds(int nw) { return nw * kLineStride<U> + 2 * nw * Team<U>::N; }

// Algorithm 1's iterations in FP64 for subcarrier k of frame f, all symbols:
// wave c holds cluster c's inverse (waves past C contribute zeros) and entry
// l % N of every vector on lane l.  B_c^{-1} is Hermitian, so entry j of a
// product is sum_i conj(M_ij) q_i over the lane's rows, then over ti.  hy: this
// lane's part of H_c^H y_c of symbol 0 (HY0; formed here otherwise).  buf: the
// consensus buffer in turn, kept by the caller from one subcarrier to the next
// (a slow wave may still be reading the other one).  NW: waves of the workgroup.
template <int U, int NW, bool HY0, class INV>
__device__ __forceinline__ void fix64_iterate(const FixArgs& f, int k, const INV& inv, d2 (&hy)[Team<U>::NB], d2* lds,
                                              int& buf) {
  constexpr int N = Team<U>::N, NB = Team<U>::NB;
  const int lane = threadIdx.x & 63, u = lane % N;
  const int c = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool on = c < f.C;   // wave-uniform
  d2* line = lds + c * kLineStride<U>;
  d2* cons = lds + NW * kLineStride<U>;
  const c32* Hc = f.H + (size_t)k * f.B * U + (size_t)c * f.S * U;
  const c32* yk = f.y + (size_t)k * f.n_sym * f.B + (size_t)c * f.S;
  auto matvec = [&](d2 q) -> d2 {
    if (lane < N) line[lane] = q;
    wave_lds_sync();
    d2 acc[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[b] = dzero();
    inv.apply(acc, line, lane);
    return ti_sum<NB>(acc);
  };
#pragma unroll 1
  for (int n = 0; n < f.n_sym; ++n) {
    d2 z = dzero(), lam = dzero(), s = dzero(), yr = dzero();
    // s = prox(sum_c (z_c + lambda_c)), in cluster order on every wave
    auto consensus = [&]() {
      d2* cb = cons + buf * NW * N;
      buf ^= 1;
      if (lane < N) cb[c * N + lane] = on ? d2{z.re + lam.re, z.im + lam.im} : dzero();
      __syncthreads();
      d2 w = cb[u];
#pragma unroll
      for (int cc = 1; cc < NW; ++cc) {
        const d2 v = cb[cc * N + u];
        w.re += v.re;
        w.im += v.im;
      }
      s = prox64(f, w);
    };
    if (on) {
      if (!HY0 || n > 0) team_hy<U>(Hc, yk + (size_t)n * f.B, f.S, lane, hy);
      yr = matvec(ti_sum<NB>(hy));   // y_c^reg = B_c^{-1} H_c^H y_c
      z = yr;
    }
    consensus();
#pragma unroll 1
    for (int t = 2; t <= f.T; ++t) {
      if (on) {
        // lambda_c += gamma (z_c - s);  z_c = y_c^reg + rho B_c^{-1} (s - lambda_c)
        lam.re = fma(f.gamma, z.re - s.re, lam.re);
        lam.im = fma(f.gamma, z.im - s.im, lam.im);
        const d2 bq = matvec(d2{s.re - lam.re, s.im - lam.im});
        z = d2{fma(f.rho, bq.re, yr.re), fma(f.rho, bq.im, yr.im)};
      }
      consensus();
    }
    if (c == 0 && lane < U) write_out(f, k, n, lane, s);
  }
}

// Algorithm 1 in FP64 for subcarrier k of frame f, U <= 32, in one workgroup.
template <int U, int NW>
__device__ __forceinline__ void fix64_subcarrier(const FixArgs& f, int k, d2* lds, int& buf) {
  const int lane = threadIdx.x & 63, c = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  RegInverse<U> inv;
  d2 hy[Team<U>::NB];
  if (c < f.C) {
    // (16 waves leave 128 registers: with four groups of rows in flight 190 spilled,
    // with two 96; B = 1536, U = 32, C = 16, 16 flagged subcarriers 158 -> 145 us)
    team_gram<U, true, (U == 32 && NW == 16) ? 2 : 4>(f.H + (size_t)k * f.B * U + (size_t)c * f.S * U,
                       f.y + (size_t)k * f.n_sym * f.B + (size_t)c * f.S, f.S, f.rho, 0, lane, inv.M, hy);
    team_invert<U>(inv.M, 0, lane, lds + c * Team<U>::kLds);
  }
  fix64_iterate<U, NW, true>(f, k, inv, hy, lds, buf);
}

// ---------------------------------------------------------------------------
// U = 64 (at most eight clusters): inverses through the workspace slot.
// ---------------------------------------------------------------------------
constexpr int kIter64 = 512;   // threads of the workgroups that iterate at U = 64

__device__ __forceinline__ void store_block64(const Tiles<64>& M, d2* Mc, int tw, int lane) {
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) Mc[tw * kBlk64 + (4 * a + b) * 64 + lane] = d2{M.re[0][b][a], M.im[0][b][a]};
}

__device__ __forceinline__ void iterate64(const FixArgs& f, int k, const d2* Ms, d2* lds, int& buf) {
  const int lane = threadIdx.x & 63, c = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  SlotInverse inv;
  if (c < f.C) inv.load(Ms + (size_t)c * 4 * kBlk64, lane);
  d2 hy[4];
  fix64_iterate<64, kIter64 / 64, false>(f, k, inv, hy, lds, buf);
}

// One whole subcarrier by a workgroup of kIter64 threads: two teams invert two
// clusters at a time into the slot, then the iterations.
__device__ __forceinline__ void fix64_subcarrier64(const FixArgs& f, int k, d2* Ms, d2* lds, int& buf) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int team = wave >> 2, tw = wave & 3;
  const c32* Hk = f.H + (size_t)k * f.B * 64;
  __syncthreads();   // the previous subcarrier's operand lines are no longer read
#pragma unroll 1
  for (int cb = 0; cb < f.C; cb += kIter64 / 256) {
    // (a team past C inverts the last cluster again and stores nothing)
    const int c = cb + team < f.C ? cb + team : f.C - 1;
    Tiles<64> M;
    d2 hy[4];
    team_gram<64, false>(Hk + (size_t)c * f.S * 64, nullptr, f.S, f.rho, tw, lane, M, hy);
    team_invert<64>(M, tw, lane, lds + team * Team<64>::kLds);
    if (cb + team < f.C) store_block64(M, Ms + (size_t)c * 4 * kBlk64, tw, lane);
  }
  __syncthreads();   // inverses in the slot
  iterate64(f, k, Ms, lds, buf);
}

}  // namespace

// The whole re-slice of one call's (or a batch's) flagged subcarriers, U <= 32.
template <int U, int NW, class FR>
__device__ __forceinline__ void admm_ul_fix64_body(const FR& fr) {
  const unsigned act = flagged_frames(fr);
  if (!act) return;   // uniform
  __shared__ FixList list;
  extern __shared__ d2 fsm[];
  int buf = 0;
  for_flagged(fr, act, gridDim.x, blockIdx.x, 0, list,
              [&](const FixArgs& f, int k) { fix64_subcarrier<U, NW>(f, k, fsm, buf); });
}

// NW: waves of the workgroup, 8 (C <= 8; twice the registers) or 16.
template <int U, int NW>
__global__ void __launch_bounds__(64 * NW) admm_ul_fix64(FixArgs f) {
  admm_ul_fix64_body<U, NW>(OneFrame{f});
}
template <int U, int NW>
__global__ void __launch_bounds__(64 * NW) admm_ul_fix64_batch(FixBatch b) {
  admm_ul_fix64_body<U, NW>(ManyFrames{b});
}

// U = 64, step 1: workgroup (c, g) forms and inverts cluster c's regularised
// Gram of the flagged subcarrier of rank g into slot g (list0[g] takes its
// index, -1 for none).  The clusters of the first ranks come first in the
// launch: with few flagged subcarriers the workgroups that have work start at
// once, not behind the ones that only scan.  The extra workgroup (0, n_slots)
// only counts: it tells step 2 whether more than n_slots subcarriers are flagged.
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) admm_ul_factor64(FixArgs f) {
  if (nothing_flagged(f)) return;   // uniform
  __shared__ FixList list;
  __shared__ d2 lds[Team<64>::kLds];
  const int G = f.n_slots, g = blockIdx.y, c = blockIdx.x;
  const OneFrame fr{f};
  const bool counting = g == G;
  if (counting && c) return;
  const long chunks = fix_chunks(fr, 1u);
  int k = -1;
  long seen = 0;
  const int wt = blockDim.x >> 6;
  for (long c0 = 0; c0 < chunks; c0 += wt) {
    // rank g of the call is rank g - seen of this window (the stride keeps the
    // list to that one entry)
    constexpr int kNone = 1 << 30;
    const long want = (long)g - seen;   // >= 0: the loop ends once it is found
    int total = 0;
    const int nl = collect_window(fr, 1u, c0, wt, list, &total,
                                  [&](int) { return Share{kNone, counting || want > kNone ? kNone : (int)want}; });
    if (nl > 0) k = list.k[0];
    seen += total;
    if (counting ? seen > G : k >= 0) break;   // uniform
  }
  if (counting) {
    if (threadIdx.x == 0) *f.more = seen > G ? 1u : 0u;
    return;
  }
  if (c == 0 && threadIdx.x == 0) f.list0[g] = k;
  if (k < 0) return;   // uniform
  const int lane = threadIdx.x & 63, tw = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  Tiles<64> M;
  d2 hy[4];
  team_gram<64, false>(f.H + (size_t)k * f.B * 64 + (size_t)c * f.S * 64, nullptr, f.S, f.rho, tw, lane, M, hy);
  team_invert<64>(M, tw, lane, lds);
  store_block64(M, static_cast<d2*>(f.ws) + ((size_t)g * f.C + c) * 4 * kBlk64, tw, lane);
}

// U = 64, step 2: the iterations of subcarrier list0[g] with the inverses of
// slot g, then this workgroup's share of the subcarriers past the first n_slots.
__global__ void __launch_bounds__(kIter64) admm_ul_iter64(FixArgs f) {
  if (nothing_flagged(f)) return;   // uniform
  __shared__ FixList list;
  extern __shared__ d2 fsm[];
  const int G = f.n_slots, g = blockIdx.x;
  d2* Ms = static_cast<d2*>(f.ws) + (size_t)g * f.C * 4 * kBlk64;
  const int k0 = f.list0[g];
  int buf = 0;
  if (k0 >= 0) iterate64(f, k0, Ms, fsm, buf);
  if (*f.more == 0u) return;   // uniform
  for_flagged(OneFrame{f}, 1u, G, g, G, list, [&](const FixArgs& fa, int k) { fix64_subcarrier64(fa, k, Ms, fsm, buf); });
}

// U = 64, a batch of frames: every flagged subcarrier by one workgroup.
__global__ void __launch_bounds__(kIter64) admm_ul_fix64_batch64(FixBatch b) {
  const ManyFrames fr{b};
  const unsigned act = flagged_frames(fr);
  if (!act) return;   // uniform
  __shared__ FixList list;
  extern __shared__ d2 fsm[];
  int buf = 0;
  for_flagged(fr, act, gridDim.x, blockIdx.x, 0, list, [&](const FixArgs& f, int k) {
    fix64_subcarrier64(f, k, static_cast<d2*>(f.ws) + (size_t)blockIdx.x * b.slot_c * 4 * kBlk64, fsm, buf);
  });
}

// Largest B U (complex entries of H[k]) the CG pass keeps in LDS (16 KiB:
// the pass's LDS stays under 64 KiB).
constexpr int kCgStage = 2048;

// Sum over the first wave of v (lanes past the data pass 0); lane 0 stores
// it at *out.  Every thread of the workgroup must call (it ends with a barrier).
__device__ __forceinline__ void wave0_sum(double v, double* out) {
  if (threadIdx.x < 64) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    if (threadIdx.x == 0) *out = v;
  }
  __syncthreads();
}

// Algorithm 2 in FP64 for the flagged subcarriers (f.rho = N0 / Es, or 0 for
// ZF).  H[k] is staged in LDS when it fits.  w = sum_c H_c^H (H_c p): H p for
// all B rows by one thread per row (blocks of 1024 rows for larger B), then
// one partial sum per (cluster, user) and the sum over the clusters in
// cluster order; the inner products by the first wave.
__global__ void __launch_bounds__(kFixThreads) dcg_ul_fix64(FixArgs f) {
  if (nothing_flagged(f)) return;   // uniform
  extern __shared__ d2 fsm[];
  constexpr int kChunk = 1024;
  const int U = f.U, C = f.C, S = f.S, B = f.B, CU = C * U;
  d2* R = fsm;
  d2* P = R + U;
  d2* X = P + U;
  d2* W = X + U;
  d2* Hp = W + U;                // kChunk entries: H_c p for a block of rows
  d2* Wp = Hp + kChunk;          // [C][U] per-cluster partial sums
  c32* Hs = reinterpret_cast<c32*>(Wp + CU);   // H[k] when B U <= kCgStage
  double* red = reinterpret_cast<double*>(Hs + kCgStage);   // [0] rr, [1] pe, [2] rr_new
  __shared__ FixList list;
  const int tid = threadIdx.x;
  const bool staged = B * U <= kCgStage;

  // w = sum_c H_c^H v_c, with v the B entries at vb (stride vs) or, when
  // vb is null, Hp: per-cluster partial sums by C U threads, then the sum
  // over the clusters in cluster order.  Ends with a barrier.
  auto hh_sum = [&](const c32* rows, const c32* yv, d2* out) {
    for (int e = tid; e < CU; e += kFixThreads) {
      const int c = e / U, i = e - c * U;
      d2 acc = dzero();
#pragma unroll 4
      for (int s = 0; s < S; ++s) {
        const int j = c * S + s;
        dmacc(acc, dld(rows + (size_t)j * U + i), yv ? dld(yv + j) : Hp[j]);
      }
      Wp[e] = acc;
    }
    __syncthreads();
    for (int i = tid; i < U; i += kFixThreads) {
      d2 acc = dzero();
      for (int c = 0; c < C; ++c) {
        acc.re += Wp[c * U + i].re;
        acc.im += Wp[c * U + i].im;
      }
      out[i] = acc;
    }
    __syncthreads();
  };

  // While workgroups outnumber a window's flagged subcarriers, `split` of them
  // share the symbols of one (nothing but the load of H[k] is repeated): without,
  // one subcarrier of 17 symbols takes 17 times as long as one of one; with a fixed
  // split 700 flagged subcarriers of three symbols (U = 16, S = 48) took 486 us
  // instead of 423.
  int split = 1, n0 = 0;
  auto recompute = [&](int k) {
    const c32* Hk = f.H + (size_t)k * B * U;
    if (staged) {
      for (int e = tid; e < B * U; e += kFixThreads) Hs[e] = Hk[e];
      __syncthreads();
    }
    const c32* rows = staged ? Hs : Hk;
    for (int n = n0; n < f.n_sym; n += split) {
      const c32* yk = f.y + ((size_t)k * f.n_sym + n) * B;
      // y^MRC = sum_c H_c^H y_c; r = p = y^MRC; x = 0
      hh_sum(rows, yk, R);
      for (int i = tid; i < U; i += kFixThreads) {
        P[i] = R[i];
        X[i] = dzero();
      }
      wave0_sum(tid < U ? R[tid].re * R[tid].re + R[tid].im * R[tid].im : 0.0, red);
      for (int t = 1; t <= f.T; ++t) {
        const double rr = red[0];
        if (rr == 0.0) break;   // uniform: every thread read the same value
        // H p for all B rows (blocks of kChunk rows when B is larger), then w = sum_c H_c^H (H_c p)
        if (B <= kChunk) {
          for (int j = tid; j < B; j += kFixThreads) {
            d2 acc = dzero();
#pragma unroll 4
            for (int u = 0; u < U; ++u) dmac(acc, dld(rows + (size_t)j * U + u), P[u]);
            Hp[j] = acc;
          }
          __syncthreads();
          hh_sum(rows, nullptr, W);
        } else {
          for (int i = tid; i < U; i += kFixThreads) W[i] = dzero();
          __syncthreads();
          for (int c = 0; c < C; ++c) {
            for (int s0 = 0; s0 < S; s0 += kChunk) {
              const int ns = (S - s0 < kChunk) ? S - s0 : kChunk;
              for (int s = tid; s < ns; s += kFixThreads) {
                const c32* row = rows + ((size_t)c * S + s0 + s) * U;
                d2 acc = dzero();
#pragma unroll 4
                for (int u = 0; u < U; ++u) dmac(acc, dld(row + u), P[u]);
                Hp[s] = acc;
              }
              __syncthreads();
              for (int i = tid; i < U; i += kFixThreads) {
                d2 acc = dzero();
#pragma unroll 4
                for (int s = 0; s < ns; ++s) dmacc(acc, dld(rows + ((size_t)c * S + s0 + s) * U + i), Hp[s]);
                W[i].re += acc.re;
                W[i].im += acc.im;
              }
              __syncthreads();
            }
          }
        }
        // e = rho p + w (kept in W); alpha = ||r||^2 / Re(p^H e)
        for (int i = tid; i < U; i += kFixThreads) W[i] = d2{f.rho * P[i].re + W[i].re, f.rho * P[i].im + W[i].im};
        __syncthreads();
        wave0_sum(tid < U ? P[tid].re * W[tid].re + P[tid].im * W[tid].im : 0.0, red + 1);
        const double alpha = rr / red[1];
        for (int i = tid; i < U; i += kFixThreads) {
          X[i] = d2{X[i].re + alpha * P[i].re, X[i].im + alpha * P[i].im};
          R[i] = d2{R[i].re - alpha * W[i].re, R[i].im - alpha * W[i].im};
        }
        __syncthreads();
        wave0_sum(tid < U ? R[tid].re * R[tid].re + R[tid].im * R[tid].im : 0.0, red + 2);
        const double rr_new = red[2];
        const double beta = rr_new / rr;
        for (int i = tid; i < U; i += kFixThreads) P[i] = d2{R[i].re + beta * P[i].re, R[i].im + beta * P[i].im};
        __syncthreads();
        if (tid == 0) red[0] = rr_new;
        __syncthreads();
      }
      for (int i = tid; i < U; i += kFixThreads) write_out(f, k, n, i, X[i]);
      __syncthreads();
    }
  };
  const OneFrame fr{f};
  const int grid = gridDim.x, wt = fix_window(blockDim.x >> 6, grid);
  const long chunks = fix_chunks(fr, 1u);
  long seen = 0;
  for (long c0 = 0; c0 < chunks; c0 += wt) {
    int total = 0, G = grid, q0 = 0;
    const int nl = collect_window(fr, 1u, c0, wt, list, &total, [&](int flagged) {
      split = min(min(f.n_sym, 16), max(1, grid / max(1, flagged)));
      G = grid / split;
      const int g = blockIdx.x / split;
      n0 = blockIdx.x % split;
      q0 = g < G ? (int)(((long)g - seen % G + G) % G) : flagged;   // (a remainder of the grid: nothing)
      return Share{G, q0};
    });
    for (int q = 0; q < nl; ++q) recompute(__builtin_amdgcn_readfirstlane(list.k[q]));
    seen += total;
  }
}

size_t fix64_slot_bytes(int U, int C) { return (size_t)C * U * U * sizeof(d2); }

template <int U, typename Args>
static void launch_fix(void (*k8)(Args), void (*k16)(Args), const Args& a, int C, unsigned grid, hipStream_t st) {
  const int nw = C <= 8 ? 8 : 16;
  hipLaunchKernelGGL(nw == 8 ? k8 : k16, dim3(grid), dim3(64 * nw), fix_lds<U>(nw) * sizeof(d2), st, a);
}

static_assert(2 * Team<64>::kLds <= fix_lds<64>(kIter64 / 64), "two teams' panels exceed the iterations' LDS");
constexpr size_t kLds64 = fix_lds<64>(kIter64 / 64) * sizeof(d2);

hipError_t launch_admm_ul_fix64(const FixArgs& f, hipStream_t st) {
  const unsigned grid = (unsigned)f.n_slots;
  switch (f.U) {
    case 8: launch_fix<8>(admm_ul_fix64<8, 8>, admm_ul_fix64<8, 16>, f, f.C, grid, st); break;
    case 16: launch_fix<16>(admm_ul_fix64<16, 8>, admm_ul_fix64<16, 16>, f, f.C, grid, st); break;
    case 32: launch_fix<32>(admm_ul_fix64<32, 8>, admm_ul_fix64<32, 16>, f, f.C, grid, st); break;
    case 64:
      hipLaunchKernelGGL(admm_ul_factor64, dim3((unsigned)f.C, grid + 1), dim3(256), 0, st, f);
      hipLaunchKernelGGL(admm_ul_iter64, dim3(grid), dim3(kIter64), kLds64, st, f);
      break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_admm_ul_fix64_batch(const FixBatch& b, int U, int n_slots, hipStream_t st) {
  if (b.n < 1) return hipSuccess;
  // U <= 32 keeps no state in the workspace: a workgroup per subcarrier up to
  // the most that a call uses
  long sc = 0;
  for (int i = 0; i < b.n; ++i) sc += b.f[i].n_sc;
  const unsigned grid = (unsigned)(sc < kFixMaxSlots ? (sc > 0 ? sc : 1) : kFixMaxSlots);
  switch (U) {
    case 8: launch_fix<8>(admm_ul_fix64_batch<8, 8>, admm_ul_fix64_batch<8, 16>, b, b.slot_c, grid, st); break;
    case 16: launch_fix<16>(admm_ul_fix64_batch<16, 8>, admm_ul_fix64_batch<16, 16>, b, b.slot_c, grid, st); break;
    case 32: launch_fix<32>(admm_ul_fix64_batch<32, 8>, admm_ul_fix64_batch<32, 16>, b, b.slot_c, grid, st); break;
    case 64:
      hipLaunchKernelGGL(admm_ul_fix64_batch64, dim3((unsigned)n_slots), dim3(kIter64), kLds64, st, b);
      break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_dcg_ul_fix64(const FixArgs& f, hipStream_t st) {
  const size_t lds = (size_t)(4 * f.U + 1024 + f.C * f.U) * sizeof(d2) + kCgStage * sizeof(c32) + 4 * sizeof(double);
  // a workgroup per (subcarrier, symbol) up to the most that a call uses
  const long items = (long)f.n_sc * f.n_sym;
  const unsigned grid = (unsigned)(items < kFixMaxSlots ? items : kFixMaxSlots);
  hipLaunchKernelGGL(dcg_ul_fix64, dim3(grid), dim3(kFixThreads), lds, st, f);
  return hipGetLastError();
}

}  // namespace dbp
