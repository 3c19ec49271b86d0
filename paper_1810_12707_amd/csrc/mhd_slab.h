// Fused z and y passes of the small grids.
//
// A workgroup owns the whole (z, y) plane of one kx of one field in LDS and runs
// its z and its y transforms back to back, so the I_z intermediate and half the
// launches of the column passes disappear.  These sizes are bound by their
// launches (about 4 us each in a replayed graph, whatever they do) and by the
// latency of one work item, not by bandwidth.  FP32 step, pass by pass -> fused
// (five launches instead of eleven: k_zyinv, the velocity pass, k_strain_rho, the flux
// pass, k_yzrhs; a sixth, k_yzfwd, with the Laplacian viscous force): 16^3 45 -> 28 us, 24^3 50 -> 34, 32^3 52 -> 40;
// batches of 16 and 64 members of 32^3 141 -> 121 and 421 -> 393 us.  At 48^3 and
// 64^3 one CU's share of the work outweighs the launches saved (59 -> 66 and 79 ->
// 97 us), so the line is at 32.
//
// LDS layout: [z][y] with a pitch of N + 1 elements, lanes along ky in the z
// transforms (unit stride) and along z in the y transforms (odd stride): both
// free of bank conflicts.  A transform that takes its input from the slab it
// works in reads all of it into registers, then a barrier, then runs in place.
//
// The transforms, multipliers and epilogues are those of k_col, k_zfwd_rhs and
// k_rho_rhs, element for element in the same order, so the results are the same
// bits.
#pragma once

#include "mhd_kernels.h"

namespace mhd {
MHD_SCHED_BEGIN

// Threads of one transform team: one first-pass butterfly each, at most 256.
template <typename T, int N> constexpr int slab_threads() {
  constexpr int w = N * (N / PlanOf<N>::r[0]);
  return w >= 256 ? 256 : (w + 63) / 64 * 64;
}
constexpr int kTeams = 3;  // transforms side by side in k_strain_rho and k_yzrhs

template <typename T, int N> struct Slab {
  using PL = PlanOf<N>;
  static constexpr int NT = slab_threads<T, N>();
  static constexpr int P = N + 1;  // pitch of a z row
  static constexpr int NB = Band<N>::NB, NH = Band<N>::NH, NHP = Band<N>::NHP;
  static constexpr int PY = Pitch<T, N>::Y;
  static constexpr int SZ = N * P;

  // Transform of NSEQ sequences by NT threads (tid 0 .. NT - 1), element (b, l) at
  // b * BS + l * ES of buf; SYNC: load() reads buf itself.  store() may write
  // position (b, pos) of buf.  Every team of a workgroup calls it together.
  template <int S, int NSEQ, int ES, int BS, bool SYNC, int NT = Slab::NT, class Load, class Store>
  static __device__ __forceinline__ void fft(cx<T>* buf, const cx<T>* stw, int tid, Load&& load, Store&& store) {
    using FP = FirstPass<PL, NSEQ, NT, 0>;
    cx<T> v[FP::CNT][FP::R];
#pragma unroll
    for (int i = 0; i < FP::CNT; ++i) {
      const int w = tid + i * NT;
      int b, j;
      lane_map<NSEQ, FP::NBF, 0>(w, b, j);
      const bool ok = FP::TOT % NT == 0 || w < FP::TOT;
#pragma unroll
      for (int r = 0; r < FP::R; ++r) v[i][r] = ok ? load(i, r, b, j + r * FP::NBF) : mk<T>(0, 0);
    }
    if constexpr (SYNC) __syncthreads();
    fft_first_regs<T, PL, NSEQ, NT, ES, BS, S, 0, 0>(buf, v, tid, NSEQ, store);
    fft_rest<T, PL, NSEQ, NT, ES, BS, S, 0, 0>(buf, stw, tid, NSEQ, store);
  }

  // y transform (forward) of plane kx of an I_y field; put(z, y, value) may write
  // position (z, y) of buf.
  template <class Put>
  static __device__ __forceinline__ void yfwd(cx<T>* buf, const cx<T>* stw, int tid, const T* src, int kx, T coef,
                                              Put&& put) {
    fft<-1, N, 1, P, false>(
        buf, stw, tid, [&](int, int, int z, int y) { return cscale(ld(src, (int64_t)(z * N + y) * PY + kx), coef); },
        [&](int, int, int z, int y, cx<T> val) { put(z, y, val); });
  }
  // y transform (inverse) of the slab in buf (column b holds ky band index b) to
  // plane kx of an I_y field.
  template <int NT = Slab::NT>
  static __device__ __forceinline__ void yinv(cx<T>* buf, const cx<T>* stw, int tid, T* dst, int kx) {
    fft<1, N, 1, P, true, NT>(
        buf, stw, tid,
        [&](int, int, int z, int y) {
          const int l = pos_band<N>(y);
          return l >= 0 ? buf[z * P + l] : mk<T>(0, 0);
        },
        [&](int, int, int z, int y, cx<T> val) { st(dst, (int64_t)(z * N + y) * PY + kx, val); });
  }
};

// Work item of a slab launch: (member, field, kx), kx fastest and XCD-blocked, so
// that the planes that share memory lines run on one XCD.
struct SlabItem {
  int m, f, kx;
};
template <int NH> __device__ __forceinline__ SlabItem slab_item(int nfields) {
  const int w = xcd_remap(blockIdx.x, gridDim.x);
  SlabItem it;
  it.m = w / (nfields * NH);
  const int rest = w - it.m * nfields * NH;
  it.f = rest / NH;
  it.kx = rest - it.f * NH;
  return it;
}

// sum of term t of sp into acc: coef * (i k_axis or 1) * x, as k_col combines it
template <typename T>
__device__ __forceinline__ void add_term(cx<T>& acc, const Term& t, cx<T> x, int kx, int ky, int kz) {
  const T cf = T(t.coef);
  if (t.axis < 0) {
    acc = cfma(cf, x, acc);
  } else {
    const T ck = cf * T(t.axis == 0 ? kx : (t.axis == 1 ? ky : kz));
    acc = cfma(ck, ctimes_i(x), acc);
  }
}

// Inverse z and y passes: compact spectra -> I_y planes.
template <typename T, int N>
__global__ void __launch_bounds__((slab_threads<T, N>())) k_zyinv(const ColArgs<T> a) {
  using SL = Slab<T, N>;
  __shared__ cx<T> buf[SL::SZ];
  __shared__ cx<T> stw[N];
  const int tid = threadIdx.x;
  const SlabItem it = slab_item<SL::NH>(a.nout);
  const OutSpec& sp = a.spec[it.f];
  load_twiddles<T, typename SL::PL, SL::NT>(stw, a.tw, tid);
  using FP = FirstPass<typename SL::PL, SL::NB, SL::NT, 0>;
  // every load of a term goes out before any is used
  cx<T> x[kMaxTerms][FP::CNT][FP::R];
#pragma unroll
  for (int t = 0; t < kMaxTerms; ++t) {
    if (t >= sp.nterms) break;
    const T* const src = member_ptr(a.in[sp.t[t].src], it.m, a.bt.mstride);
#pragma unroll
    for (int i = 0; i < FP::CNT; ++i) {
      const int w = tid + i * SL::NT;
      int b, j;
      lane_map<SL::NB, FP::NBF, 0>(w, b, j);
#pragma unroll
      for (int r = 0; r < FP::R; ++r) {
        const int l = pos_band<N>(j + r * FP::NBF);
        const bool ok = (FP::TOT % SL::NT == 0 || w < FP::TOT) && l >= 0;
        x[t][i][r] = ok ? ld(src, (int64_t)(l * SL::NB + b) * SL::NHP + it.kx) : mk<T>(0, 0);
      }
    }
  }
  SL::template fft<1, SL::NB, SL::P, 1, false>(
      buf, stw, tid,
      [&](int i, int r, int b, int q) {
        cx<T> acc = mk<T>(0, 0);
        const int l = pos_band<N>(q);
        if (l < 0) return acc;
#pragma unroll
        for (int t = 0; t < kMaxTerms; ++t)
          if (t < sp.nterms) add_term<T>(acc, sp.t[t], x[t][i][r], it.kx, band_k<N>(b), band_k<N>(l));
        return acc;
      },
      [&](int, int, int b, int q, cx<T> val) { buf[q * SL::P + b] = val; });
  __syncthreads();
  SL::yinv(buf, stw, tid, member_ptr(a.out[it.f], it.m, a.bt.mstride), it.kx);
}

// Forward y and z passes: I_y planes (row-pass outputs, doubled: halved here) ->
// compact spectra.
template <typename T, int N>
__global__ void __launch_bounds__((slab_threads<T, N>())) k_yzfwd(const ColArgs<T> a) {
  using SL = Slab<T, N>;
  __shared__ cx<T> buf[SL::SZ];
  __shared__ cx<T> stw[N];
  const int tid = threadIdx.x;
  const SlabItem it = slab_item<SL::NH>(a.nout);
  load_twiddles<T, typename SL::PL, SL::NT>(stw, a.tw, tid);
  SL::yfwd(buf, stw, tid, member_ptr(a.in[it.f], it.m, a.bt.mstride), it.kx, T(0.5),
           [&](int z, int y, cx<T> val) { buf[z * SL::P + y] = val; });
  __syncthreads();
  T* const out = member_ptr(a.out[it.f], it.m, a.bt.mstride);
  SL::template fft<-1, SL::NB, SL::P, 1, true>(
      buf, stw, tid, [&](int, int, int b, int z) { return buf[z * SL::P + band_pos<N>(b)]; },
      [&](int, int, int b, int q, cx<T> val) {
        const int l = pos_band<N>(q);
        if (l >= 0) st(out, (int64_t)(l * SL::NB + b) * SL::NHP + it.kx, val);
      });
}

// Velocity planes -> strain planes: forward y and z of the components a strain
// needs, their spectral combination, inverse z and y.  The components (up to three)
// are transformed side by side by one team of threads each, so that a workgroup's
// chain is four transforms long; each is transformed once per strain that uses it
// (12 planes of work instead of 3, on a chip that is nearly idle at these sizes,
// against a launch and a pass through memory).  Field a.nout is the density
// right-hand side and update, which needs m^ before the last pass of the step
// overwrites it.
template <typename T, int N>
__global__ void __launch_bounds__((kTeams * slab_threads<T, N>()))
    k_strain_rho(const ColArgs<T> a, const UpdateArgs<T> q) {
  using SL = Slab<T, N>;
  constexpr int NT = SL::NT, NA = kTeams * NT;
  __shared__ cx<T> buf[kTeams][SL::SZ];
  __shared__ cx<T> stw[N];
  const int tid = threadIdx.x, team = __builtin_amdgcn_readfirstlane(tid / NT), ttid = tid - team * NT;
  const SlabItem it = slab_item<SL::NH>(a.nout + 1);
  if (it.f == a.nout) {
    for (int e = tid; e < SL::NB * SL::NB; e += NA) {
      const int l = e / SL::NB, b = e - l * SL::NB;
      rho_entry<T>(q, it.m, (int64_t)e * SL::NHP + it.kx, it.kx, band_k<N>(b), band_k<N>(l));
    }
    return;
  }
  const OutSpec& sp = a.spec[it.f];
  load_twiddles<T, typename SL::PL, NA>(stw, a.tw, tid);
  // a team without a term of its own repeats the last one (its result is not read)
  const int mine = team < sp.nterms ? team : sp.nterms - 1;
  cx<T>* const own = buf[team];
  SL::yfwd(own, stw, ttid, member_ptr(a.in[sp.t[mine].src], it.m, a.bt.mstride), it.kx, T(0.5),
           [&](int z, int y, cx<T> val) { own[z * SL::P + y] = val; });
  __syncthreads();
  SL::template fft<-1, SL::NB, SL::P, 1, true>(
      own, stw, ttid, [&](int, int, int b, int z) { return own[z * SL::P + band_pos<N>(b)]; },
      [&](int, int, int b, int p, cx<T> val) { own[p * SL::P + b] = val; });
  __syncthreads();
  SL::template fft<1, SL::NB, SL::P, 1, true, NA>(
      buf[0], stw, tid,
      [&](int, int, int b, int p) {
        cx<T> acc = mk<T>(0, 0);
        const int l = pos_band<N>(p);
        if (l < 0) return acc;
#pragma unroll
        for (int t = 0; t < kTeams; ++t)
          if (t < sp.nterms) add_term<T>(acc, sp.t[t], buf[t][p * SL::P + b], it.kx, band_k<N>(b), band_k<N>(l));
        return acc;
      },
      [&](int, int, int b, int p, cx<T> val) { buf[0][p * SL::P + b] = val; });
  __syncthreads();
  SL::template yinv<NA>(buf[0], stw, tid, member_ptr(a.out[it.f], it.m, a.bt.mstride), it.kx);
}

// Flux planes -> right-hand sides and update of m, B and E (fields 1..7): forward y
// of the up to three fluxes side by side (teams 0, 1: the terms of A_f, team 2:
// Z_f), forward z of their combinations, and the epilogue of k_zfwd_rhs over all
// threads.  The nfrozen fields after them are those a kinematic run freezes.
template <typename T, int N>
__global__ void __launch_bounds__((kTeams * slab_threads<T, N>()))
    k_yzrhs(const RhsArgs<T> a, int nfrozen) {
  using SL = Slab<T, N>;
  constexpr int NT = SL::NT, NA = kTeams * NT;
  constexpr int NE = SL::NB * SL::NB, CNT = (NE + NA - 1) / NA;  // entries of this kx, per thread
  __shared__ cx<T> buf[kTeams][SL::SZ];
  __shared__ cx<T> stw[N];
  const int tid = threadIdx.x, team = __builtin_amdgcn_readfirstlane(tid / NT), ttid = tid - team * NT;
  const SlabItem it = slab_item<SL::NH>(a.nf + nfrozen);
  if (it.f >= a.nf) {
    for (int e = tid; e < NE; e += NA) frozen_entry<T>(a.up, it.m, it.f - a.nf, (int64_t)e * SL::NHP + it.kx);
    return;
  }
  const int f = it.f + a.f0;
  const OutSpec& A = a.A[f];
  const OutSpec& Z = a.Z[f];
  // the state and the history, in flight during the transforms
  const RhsMember<T> M(a, it.m, f);
  cx<T> u[CNT], rp[CNT];
#pragma unroll
  for (int i = 0; i < CNT; ++i) {
    const int e = tid + i * NA;
    const int64_t off = (int64_t)e * SL::NHP + it.kx;
    u[i] = e < NE ? M.up.old_u(off) : mk<T>(0, 0);
    rp[i] = e < NE ? M.up.old_acc(off) : mk<T>(0, 0);
  }
  load_twiddles<T, typename SL::PL, NA>(stw, a.tw, tid);
  // a team without a term of its own repeats A's first (its result is not read)
  const int src = team == 2 ? (Z.nterms > 0 ? Z.t[0].src : A.t[0].src) : A.t[team < A.nterms ? team : 0].src;
  cx<T>* const own = buf[team];
  SL::yfwd(own, stw, ttid, member_ptr(a.flux[src], it.m, a.up.bt.mstride), it.kx, T(0.5),
           [&](int z, int y, cx<T> val) { own[z * SL::P + y] = val; });
  __syncthreads();
  SL::template fft<-1, SL::NB, SL::P, 1, true>(
      own, stw, ttid,
      [&](int, int, int b, int z) {
        const int at = z * SL::P + band_pos<N>(b);
        cx<T> v = mk<T>(0, 0);
        if (team == 2) {
          if (Z.nterms > 0) add_term<T>(v, Z.t[0], own[at], it.kx, band_k<N>(b), 0);
        } else if (team == 0) {
          add_term<T>(v, A.t[0], own[at], it.kx, band_k<N>(b), 0);
          if (A.nterms > 1) add_term<T>(v, A.t[1], buf[1][at], it.kx, band_k<N>(b), 0);
        }
        return v;
      },
      [&](int, int, int b, int p, cx<T> val) { own[p * SL::P + b] = val; });
  __syncthreads();
#pragma unroll
  for (int i = 0; i < CNT; ++i) {
    const int e = tid + i * NA;
    if (e >= NE) continue;
    const int l = e / SL::NB, b = e - l * SL::NB, kz = band_k<N>(l);
    const int at = band_pos<N>(l) * SL::P + b;
    cx<T> R = buf[0][at];
    if (Z.nterms > 0) R = cfma(T(kz), ctimes_i(buf[2][at]), R);
    M.apply((int64_t)e * SL::NHP + it.kx, R, u[i], rp[i], it.kx, band_k<N>(b), kz);
  }
}

MHD_SCHED_END
}  // namespace mhd
