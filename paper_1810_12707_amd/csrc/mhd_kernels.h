// Pass kernels of the pseudo-spectral MHD right-hand side, templated on the
// working precision T and the grid size N.
//
// Column passes (k_col, k_zfwd_rhs) transform along z or y for a tile of C
// adjacent columns (the contiguous kx or (ky, kx) index), so every global
// access is a run of C consecutive complex values; the tile sits in LDS as
// [N][C].  Row passes (k_row) own two adjacent x rows (z, y) and (z, y+1) of
// every field they touch: the two real rows of one field are packed as one
// complex sequence (row0 + i row1), so one length-N complex FFT does two real
// transforms, and all fields of a row pair are resident in LDS at once for the
// pointwise work.
#pragma once

#include "mhd_fft.h"
#include "mhd_internal.h"

namespace mhd {
MHD_SCHED_BEGIN

template <int N> struct Band {
  static constexpr int K = (N - 1) / 3;
  static constexpr int NH = K + 1;
  static constexpr int NB = 2 * K + 1;
  static constexpr int NHP = (NH + 7) / 8 * 8;  // kx pitch of every layout (64-byte rows)
};

// Pitches of the intermediates, in whole 128-byte lines: the kx row of I_y, and
// the z plane of I_z (whose rows keep the compact pitch NHP, so that a z pass
// over flattened (ky, kx) columns transforms no more padding than it has to).
template <typename T, int N> struct Pitch {
  static constexpr int AL = kLineBytes / (2 * (int)sizeof(T));
  static constexpr int Y = (Band<N>::NH + AL - 1) / AL * AL;
  static constexpr int Z = (Band<N>::NB * Band<N>::NHP + AL - 1) / AL * AL;
};

// Position of band index l on a length-N axis, and its wavenumber.
template <int N> __device__ __forceinline__ int band_pos(int l) { return l <= Band<N>::K ? l : l + N - Band<N>::NB; }
template <int N> __device__ __forceinline__ int band_k(int l) { return l <= Band<N>::K ? l : l - Band<N>::NB; }

// Default column tile: 16 columns while the LDS tile stays within 32 KiB,
// else 8.  The alternative schedule takes 8-column tiles (twice the work
// items, half the LDS per workgroup).
template <typename T, int N> constexpr int col_width() {
  constexpr int bytes = N * 2 * (int)sizeof(T);
  if (MHD_SCHED == 1) return 8;
  return 32768 / bytes >= 16 ? 16 : 8;
}

// Threads and tile width of the forward-z RHS pass.  It is latency-bound
// (dependent memory phases per workgroup: the first flux group, the second,
// the state and history), so it wants many resident waves and whole 128-byte row
// segments: one first-pass butterfly per thread on 16 columns from N = 256 (512
// threads; 1024 at 384 and 512: 384 FP32 924 -> 890 us, FP64 1985 -> 1656 us), 8
// columns and 1024 threads at 1024 (FP32 228 -> 106 registers: 28.0 -> 21.4 ms).  FP64
// at 512 takes 512 threads on its 8-column tiles (146 registers instead of 256 with
// 256 threads: 6.89 -> 4.35 ms).  FP32 at 192 and 96 take 8 columns and 256 threads
// (more, smaller workgroups: 126 -> 102 and 17.3 -> 16.3 us).
template <typename T, int N> constexpr bool rhs_wide() { return sizeof(T) == 4 && N >= 256; }
template <typename T, int N> constexpr int rhs_threads() {
  if (sizeof(T) == 8 && N == 512) return 2 * kThreads;
  if (N == 384 || (sizeof(T) == 4 && (N == 512 || N == 1024))) return 4 * kThreads;
  return rhs_wide<T, N>() ? 2 * kThreads : kThreads;
}
template <typename T, int N> constexpr int rhs_tile() {
  if (N == 384 || (sizeof(T) == 4 && (N == 256 || N == 512))) return 16;
  if (sizeof(T) == 4 && (N == 192 || (N == 96 && MHD_SCHED == 0))) return 8;
  return rhs_wide<T, N>() ? 8 : col_width<T, N>();
}
// Both flux groups loaded before the first is transformed, one memory phase instead
// of two, from N = 512.  With the state and history loaded after the transforms the
// kernel fits 64 registers there, so that two workgroups of 1024 threads share a CU
// and one loads while the other transforms (512 FP32: 2032 us with one workgroup of
// 94 registers -> 1650; capped without the early loads 1787; stored past the caches
// 1592, 4.6 TB/s; FP64 120 registers, 4022 -> 3290; 1024: 21.4 -> 16.8 ms).  Below,
// the second group's registers cost resident waves (256 FP32: 213 -> 279, 128: 29 ->
// 35).
template <int N> constexpr bool rhs_upfront() { return N >= 512; }
// Minimum resident waves per SIMD asked of the compiler (register cap).  FP32 from
// 512: 64 registers, as above (68 uncapped at 1024, 8 bytes of scratch capped).  A cap of
// seven waves at 128 FP32 measured nothing, for one run (28.0 us with, 28.0 without) or for
// groups of 2 to 64 (64: step 13.85 and 13.86 ms).
template <typename T, int N> constexpr int rhs_min_waves() {
  if (sizeof(T) == 4 && (N == 512 || N == 1024)) return 8;
  return rhs_wide<T, N>() || rhs_threads<T, N>() > kThreads ? 1 : 3;
}

// Threads and tile width (columns) of the column passes: S = +1 inverse, -1
// forward; MAXT input terms per element; Z axis z, else y.  Two things decide
// them, measured per pass class (microseconds per launch in the step, before ->
// after):
//  - a tile's row segment is a run of C columns, and a persistent workgroup has
//    one tile's loads in flight: wide tiles (256-byte segments, 1024 threads) keep
//    more bytes in flight per CU where the arrays come from HBM (256 FP32 12-field
//    y passes 269 -> 255 and 254 -> 239; FP64 445 -> 419), narrow ones make more
//    items for the small z launches;
//  - one first-pass butterfly per thread (fewest registers, most waves) is the
//    fastest for the inverse passes throughout and for most forward ones; the
//    three-term pass, which holds three inputs per element, only fits that way
//    (384 FP32 652 -> 492; 256 FP64 291 -> 266, with 168 bytes of scratch at its 128
//    registers; 512 FP64 3020 -> 2380).
// Sizes up to 128: 16 columns while the tile stays within 32 KiB; 128 threads at
// 64 (256 left half of them idle: step 81 -> 79).
struct ColShape {
  int c, nt;
};
template <typename T, int N, bool MX, int S, int MAXT, bool Z> constexpr ColShape col_shape() {
  constexpr bool f32 = sizeof(T) == 4, one = MAXT == 1;
  if (MHD_SCHED == 0) {
    if (N == 64 && !MX) return {16, 128};
    if (N == 192 && !MX) {
      if (f32) return !one ? ColShape{16, 512} : (S > 0 ? ColShape{32, 512} : ColShape{16, 256});
      return !one ? ColShape{8, 256} : (S > 0 ? ColShape{32, 1024} : ColShape{16, 512});
    }
    if (N == 256) {
      if (!Z || (f32 && !one)) return {32, 1024};
      return {16, f32 && !MX && S < 0 ? 256 : 512};
    }
    if (N == 384) {
      if (MX) return {16, 512};
      return f32 || one ? ColShape{16, 1024} : ColShape{8, 512};
    }
    if (N == 512) return f32 ? ColShape{16, 1024} : ColShape{8, 512};
    if (N == 768) return {8, f32 ? 512 : 256};
    if (N == 1024) return {8, 1024};
  }
  return {col_width<T, N>(), kThreads};
}
template <typename T, int N, bool MX, int S, int MAXT, bool Z> constexpr int col_threads() {
  return col_shape<T, N, MX, S, MAXT, Z>().nt;
}
template <typename T, int N, bool MX, int S, int MAXT, bool Z> constexpr int col_tile() {
  return col_shape<T, N, MX, S, MAXT, Z>().c;
}

template <typename T>
__device__ __forceinline__ cx<T> ld(const T* base, int64_t idx) {
  return reinterpret_cast<const cx<T>*>(base)[idx];
}
// Stores through a two-element vector type: stored as the struct that cx<T> is, a
// column pass's values took 8-12 more registers (192 FP32: 12-field y pass 87 ->
// 73 us, step 650 -> 630; 128: 212 -> 208).
template <typename T> using vec2 = T __attribute__((ext_vector_type(2)));
template <typename T>
__device__ __forceinline__ void st(T* base, int64_t idx, cx<T> v) {
  const vec2<T> w = {v.x, v.y};
  reinterpret_cast<vec2<T>*>(base)[idx] = w;
}

// Store past the caches (nontemporal).
template <typename T>
__device__ __forceinline__ void st_stream(T* base, int64_t idx, cx<T> v) {
  const vec2<T> w = {v.x, v.y};
  __builtin_nontemporal_store(w, reinterpret_cast<vec2<T>*>(base) + idx);
}

template <typename T, class PL, int NT>
__device__ __forceinline__ void load_twiddles(cx<T>* stw, const T* tw, int tid) {
  for (int i = tid; i < tw_entries<PL>(); i += NT) stw[i] = ld(tw, i);
}

// Band index of position q on a length-N axis, or -1 in the dropped gap.
template <int N> __device__ __forceinline__ int pos_band(int q) {
  return q <= Band<N>::K ? q : (q >= N - Band<N>::K ? q - N + Band<N>::NB : -1);
}

// Decode a flat workgroup id into (tile, field) with the field fastest, after
// the XCD remap: the outputs of one column tile run back to back on one XCD and
// share the L2 copies of the inputs they have in common.
struct TileField {
  int tile, field;
};
__device__ __forceinline__ TileField tile_field(int nfields) {
  const int L = xcd_remap(blockIdx.x, gridDim.x);
  TileField t;
  t.tile = L / nfields;
  t.field = L - t.tile * nfields;
  return t;
}

// ------------------------------------------------------------------ k_col
// S = +1: inverse pass, band (nb) in -> N out.  S = -1: forward, N in -> band out.
// Persistent: items (outer, tile, field), field fastest, walked in XCD-blocked
// order (xcd_item), so the outputs of one tile -- which share inputs -- run
// together on one XCD.  The first FFT pass reads its inputs from registers
// that were loaded from HBM while the previous item was being transformed
// (up to MAXT input terms per element; the zero gap of a band input is never
// loaded); the last pass stores straight to HBM (dropped modes skipped).
// STREAM: at 128, 256, 512 and 768 (by measurement: the strides of powers of two crowd
// into few cache sets), outputs that do not fit in the memory-side cache are stored past
// the caches: they would only displace what the next pass still finds there (256 FP32: 12-field
// inverse y pass 257 -> 203 us, forward 241 -> 221, rho pass 35 -> 27; FP64 4-field
// inverse y pass 143 -> 123; 512 FP32: 1682 -> 1560, 1563 -> 1490, 220 -> 190; 768: step
// 59.5 -> 57.0 ms).  An inverse z pass by itself may lose by it while the y pass after it
// gains more, and the three-term one gains (512 FP32, z / y: 4 fields 367 -> 391 / 554 ->
// 508 us, 12 fields 1076 -> 1089 / 1603 -> 1557, step 10.73 -> 10.67 ms; FP64 step 21.5 ->
// 21.1, mixed 10.93 -> 10.80; 768 FP32 60.0 -> 59.2); only the mixed path's one-term z
// pass at 768 has no such gain after it (1.44 -> 1.53 ms; kinematic step 18.4 -> 18.6).
// Outputs that fit stay (256 FP32, 4-field passes streamed: z 46 -> 52, y 66 -> 73), and
// so do those of the forward z pass, which the next pass reads first (512: 257 -> 273
// streamed), and of the other sizes (FP64 192: 139 -> 163 and 137 -> 150 streamed; 384:
// 1209 -> 1247 and 1193 -> 1205; 1024 FP32, 4 fields: z 3.82 -> 3.96, y 4.44 -> 4.91 and
// 3.12 -> 3.76 ms, step 107.3-109.7 -> 110.9, mixed 104.7-107.1 -> 107.5).  A launch
// chooses by its output bytes (kStreamBytes); at 512 and 768 every field list of a step
// is too large.  A branch in one kernel instead costs it 8-12 registers (192 FP32
// 12-field inverse y pass 71 -> 87 us).
// Z: a z pass (else a y pass), fixed at compile time so that the column
// geometry, the strides and the wavenumbers of the multipliers are constants
// rather than uniform branches per element.
enum ColStream { CS_NEVER, CS_BY_SIZE, CS_ALWAYS };
template <int N, int S, int MAXT, bool MX, bool Z> constexpr ColStream col_stream() {
  if (Z && S < 0) return CS_NEVER;
  if (N == 1024 || (N == 768 && MX && Z && MAXT == 1)) return CS_NEVER;
  if (N >= 512) return CS_ALWAYS;
  return is_pow2(N) && N >= 128 ? CS_BY_SIZE : CS_NEVER;
}
template <typename T, int N, int S, int MAXT, bool MX, bool Z, bool STREAM>
__global__ void __launch_bounds__((col_threads<T, N, MX, S, MAXT, Z>())) k_col(const ColArgs<T> a) {
  using PL = PlanOf<N, MX>;
  constexpr int C = col_tile<T, N, MX, S, MAXT, Z>();
  constexpr int NT = col_threads<T, N, MX, S, MAXT, Z>();
  constexpr int NH = Band<N>::NH, NHP = Band<N>::NHP, NBB = Band<N>::NB;
  using FP = FirstPass<PL, C, NT>;
  __shared__ cx<T> tile[N * C];
  __shared__ cx<T> stw[N];
  const int tid = threadIdx.x;
  constexpr bool zpass = Z;
  // z passes: columns are (ky, kx) flattened over the padded pitch; padding
  // columns (kx >= NH) are never read or written
  constexpr int ncols = zpass ? NBB * NHP : NH;
  constexpr int ntiles = (ncols + C - 1) / C;
  const int per_mem = ntiles * (zpass ? 1 : N) * a.nout;
  const int total = per_mem * a.bt.nmem;  // < 2^31 for every supported size and member count
  // strides (complex elements) of the input and output layouts: z passes
  // (either direction) map [kz][ky][kx] onto itself; the inverse y pass reads
  // [kz][ky band][kx] and writes [kz][y][kx], the forward one the reverse
  constexpr int64_t PY = Pitch<T, N>::Y, PZ = Pitch<T, N>::Z;
  constexpr int64_t os_in = zpass ? 0 : (S > 0 ? PZ : N * PY);
  constexpr int64_t ls_in = zpass ? (S > 0 ? (int64_t)NBB * NHP : PZ) : (S > 0 ? NHP : PY);
  constexpr int64_t os_out = zpass ? 0 : (S > 0 ? N * PY : PZ);
  constexpr int64_t ls_out = zpass ? (S > 0 ? PZ : (int64_t)NBB * NHP) : (S > 0 ? PY : NHP);
  load_twiddles<T, PL, NT>(stw, a.tw, tid);
  auto col_ok = [&](int col) { return col < ncols && (!zpass || col - (col / NHP) * NHP < NH); };

  struct Item {
    int m, f, outer, c0;
  };
  auto decode = [&](int item) {
    Item it;
    it.m = item / per_mem;
    const int rest = item - it.m * per_mem;
    const int t = rest / a.nout;
    it.f = rest - t * a.nout;
    it.outer = t / ntiles;
    it.c0 = (t - it.outer * ntiles) * C;
    return it;
  };
  // raw first-pass loads of one item, one set per input term
  cx<T> px[MAXT][FP::CNT][FP::R];
  auto issue = [&](const Item& it) {
    // the item's input pointers, once per item (uniform: scalar registers)
    // rather than once per element under the element's predicate
    const OutSpec& sp = a.spec[it.f];
    const int nt = sp.nterms;
    const T* src[MAXT];
#pragma unroll
    for (int t = 0; t < MAXT; ++t) src[t] = member_ptr(a.in[t < nt ? sp.t[t].src : 0], it.m, a.bt.mstride);
    const int64_t base_in = it.outer * os_in + it.c0;
#pragma unroll
    for (int i = 0; i < FP::CNT; ++i) {
      const int w = tid + i * NT;
      int c, j;
      lane_map<C, FP::NBF, 0>(w, c, j);
      const bool ok = (FP::TOT % NT == 0 || w < FP::TOT) && col_ok(it.c0 + c);
#pragma unroll
      for (int r = 0; r < FP::R; ++r) {
        const int q = j + r * FP::NBF;
        const int l = S > 0 ? pos_band<N>(q) : q;
        // the previous item's values are dead: say so, so that the compiler
        // need not keep them (and wait on loads in flight) when a load below
        // is predicated off
#pragma unroll
        for (int t = 0; t < MAXT; ++t) px[t][i][r] = mk<T>(0, 0);
        if (ok && l >= 0) {
          const int64_t idx = base_in + l * ls_in + c;
#pragma unroll
          for (int t = 0; t < MAXT; ++t)
            if (t < nt) px[t][i][r] = ld(src[t], idx);
        }
      }
    }
  };

  const int G = gridDim.x;
  int item = (int)xcd_item(blockIdx.x, G, 0, total);
  if (item >= 0) issue(decode(item));
  for (int k = 0; item >= 0; ++k) {
    const Item it = decode(item);
    // the item's multipliers, once per item
    const OutSpec& sp = a.spec[it.f];
    // Each term is re * x or dk * (i k_axis) * x.  The three-term pass and
    // the mixed path set the factor that does not apply to zero and combine
    // without a branch per element (absent terms have both zero and zeroed
    // prefetch registers): 4.6% faster for the three-term pass at 512.  The
    // FP32 and FP64 one-term passes keep the branch on the term's kind
    // (uniform), which measured faster there.
    const int nt = sp.nterms;
    T re[MAXT], dk[MAXT];
    int ax[MAXT];
#pragma unroll
    for (int t = 0; t < MAXT; ++t) {
      const int axis = t < nt ? sp.t[t].axis : -1;
      const T cf = t < nt ? T(sp.t[t].coef) : T(0);
      re[t] = axis < 0 ? cf : T(0);
      dk[t] = axis < 0 ? T(0) : cf;
      ax[t] = axis;
    }
    // combine the prefetched terms with their spectral multipliers
    cx<T> v[FP::CNT][FP::R];
#pragma unroll
    for (int i = 0; i < FP::CNT; ++i) {
      const int w = tid + i * NT;
      int c, j;
      lane_map<C, FP::NBF, 0>(w, c, j);
      const int col = it.c0 + c;
      const bool ok = (FP::TOT % NT == 0 || w < FP::TOT) && col_ok(col);
      int kx, ky = 0;
      if (zpass) {
        ky = band_k<N>(col / NHP);
        kx = col - (col / NHP) * NHP;
      } else {
        kx = col;
      }
#pragma unroll
      for (int r = 0; r < FP::R; ++r) {
        const int q = j + r * FP::NBF;
        const int l = S > 0 ? pos_band<N>(q) : q;
        cx<T> acc = mk<T>(0, 0);
        if (ok && l >= 0) {
          int kyy = ky, kz = 0;
          if (S > 0) {
            if (zpass) kz = band_k<N>(l);
            else kyy = band_k<N>(l);
          }
#pragma unroll
          for (int t = 0; t < MAXT; ++t) {
            const cx<T> xv = px[t][i][r];
            if constexpr (MAXT > 1 || MX) {
              const T ck = dk[t] * T(ax[t] == 1 ? kyy : (ax[t] == 2 ? kz : kx));
              acc.x = fma_(-ck, xv.y, fma_(re[t], xv.x, acc.x));
              acc.y = fma_(ck, xv.x, fma_(re[t], xv.y, acc.y));
            } else if (t < nt) {
              if (ax[t] < 0) {
                acc = cfma(re[t], xv, acc);
              } else {
                const T ck = dk[t] * T(ax[t] == 0 ? kx : (ax[t] == 1 ? kyy : kz));
                acc = cfma(ck, ctimes_i(xv), acc);
              }
            }
          }
        }
        v[i][r] = acc;
      }
    }
    // The next item's loads go out before this item's first pass where that
    // measured faster (FP32 forward and three-term passes from N = 256: 3-6%
    // at 512), else after it; either way they are in flight during the LDS
    // passes.
    constexpr bool EARLY = sizeof(T) == 4 && !MX && N >= 256 && (S < 0 || MAXT > 1);
    const int next = (int)xcd_item(blockIdx.x, G, k + 1, total);
    if constexpr (EARLY) {
      if (next >= 0) issue(decode(next));
    }
    __syncthreads();  // the previous item's last pass is done reading the tile
    T* out = member_ptr(a.out[it.f], it.m, a.bt.mstride);
    const int64_t base_out = it.outer * os_out + it.c0;
    auto store = [&](int, int, int c, int q, cx<T> val) {
      if (!col_ok(it.c0 + c)) return;
      int l = q;
      if constexpr (S < 0) {
        l = pos_band<N>(q);
        if (l < 0) return;
      }
      if constexpr (STREAM) st_stream(out, base_out + l * ls_out + c, val);
      else st(out, base_out + l * ls_out + c, val);
    };
    fft_first_regs<T, PL, C, NT, C, 1, S, 0, 0>(tile, v, tid, C, store);
    if constexpr (!EARLY) {
      if (next >= 0) issue(decode(next));
    }
    // mixed plans: one-term passes overlap two MFMA groups (the three-term
    // inverse pass would spill)
    fft_rest<T, PL, C, NT, C, 1, S, 0, 0, false, (MAXT == 1 ? 2 : 1)>(tile, stw, tid, C, store);
    item = next;
  }
}

// ------------------------------------------------------------------ right-hand-side epilogue
// The update of field f (0..7) of one member: see UpdateOp.  off: entry of the
// compact spectrum.
template <typename T> struct Update {
  int op;
  T *state, *u, *acc, *us, *rout;  // field f
  T dt, ac, ap, c, w;
  bool use_prev;
  __device__ __forceinline__ Update(const UpdateArgs<T>& a, int mem, int f) {
    const int64_t ms = a.bt.mstride, at = 2 * f * a.g.sc;
    op = a.op;
    state = member_ptr(a.state, mem, ms) + at;
    u = member_ptr(a.u, mem, ms) + at;
    acc = member_ptr(a.acc, mem, ms) + at;
    us = member_ptr(a.us, mem, ms) + at;
    rout = member_ptr(a.rout, mem, ms) + at;
    dt = T(a.dt[mem]);
    ac = T(a.a_cur[mem]);
    ap = T(a.a_prev[mem]);
    c = T(a.c);
    w = T(a.w);
    use_prev = a.a_prev[mem] != 0.0;
  }
  __device__ __forceinline__ bool reads_acc() const {
    return op == UP_RK_MID || op == UP_LAST || ((op == UP_AB2 || op == UP_PC_PRED) && use_prev);
  }
  __device__ __forceinline__ bool at_u() const { return op != UP_RK_MID && op != UP_LAST && op != UP_STORE; }  // U = u
  __device__ __forceinline__ cx<T> old_u(int64_t off) const { return op != UP_STORE ? ld(u, off) : mk<T>(0, 0); }
  __device__ __forceinline__ cx<T> old_acc(int64_t off) const { return reads_acc() ? ld(acc, off) : mk<T>(0, 0); }
  // u0, a0: old_u and old_acc of the entry; STREAM: store past the caches
  template <bool STREAM = false> __device__ __forceinline__ void apply(int64_t off, cx<T> R, cx<T> u0, cx<T> a0) const {
    auto put = [&](T* p, cx<T> v) {
      if constexpr (STREAM) st_stream(p, off, v);
      else st(p, off, v);
    };
    if (op == UP_STORE) {
      put(rout, R);
    } else if (op == UP_AB2 || op == UP_PC_PRED) {
      cx<T> inc = cscale(R, ac);
      if (use_prev) inc = cfma(ap, a0, inc);
      put(op == UP_AB2 ? u : us, cfma(dt, inc, u0));
      put(acc, R);
    } else if (op == UP_LAST) {
      put(u, cfma(c, cadd(a0, R), u0));
    } else {
      put(acc, op == UP_RK_FIRST ? R : cfma(w, R, a0));
      put(us, cfma(c, R, u0));
    }
  }
};

// Field f (1..7) in the last pass of a right-hand side: the resistive term, the
// Section V variants and the update.
template <typename T> struct RhsMember {
  const RhsArgs<T>& a;
  Update<T> up;
  const T *uhat, *force;  // the entries that belong to field f
  T eta;
  bool induction;
  __device__ __forceinline__ RhsMember(const RhsArgs<T>& args, int mem, int f) : a(args), up(args.up, mem, f) {
    const int64_t ms = a.up.bt.mstride, sc = a.up.g.sc;
    const int vslot = f <= 3 ? f - 1 : 3;  // u^_{f-1} for the momentum, q^ for the energy
    uhat = member_ptr(a.uhat, mem, ms) + 2 * vslot * sc;
    force = a.force ? member_ptr(a.force, mem, ms) + 2 * vslot * sc : nullptr;
    eta = T(a.eta[mem]);
    induction = f >= 4 && f <= 6;
  }
  template <bool STREAM = false>
  __device__ __forceinline__ void apply(int64_t off, cx<T> R, cx<T> u0, cx<T> a0, int kx, int ky, int kz) const {
    const T k2 = T(kx * kx + ky * ky + kz * kz);
    if (induction) {
      // MHD4 resistive term: - eta |k|^2 B^
      R = cfma(-(eta * k2), up.at_u() ? u0 : ld(up.state, off), R);
    } else {
      // viscous force mu lap u, and mu lap(|u|^2/2) in the energy
      if (a.mu != 0.0) R = cfma(-(T(a.mu) * k2), ld(uhat, off), R);
      if (a.force) R = cadd(R, ld(force, off));
    }
    up.template apply<STREAM>(off, R, u0, a0);
  }
};

// One entry of Eq. MHD1 in spectral form, R_rho = -i k . m^, and its update.
template <typename T>
__device__ __forceinline__ void rho_entry(const UpdateArgs<T>& a, int mem, int64_t idx, int kx, int ky, int kz) {
  const int64_t sc = a.g.sc;
  const T* const state = member_ptr(a.state, mem, a.bt.mstride);
  const cx<T> mx = ld(state, sc + idx), my = ld(state, 2 * sc + idx), mz = ld(state, 3 * sc + idx);
  const Update<T> up(a, mem, 0);
  const cx<T> u0 = up.old_u(idx), a0 = up.old_acc(idx);
  const cx<T> d = cfma(T(kz), mz, cfma(T(ky), my, cscale(mx, T(kx))));
  up.apply(idx, ctimes_mi(d), u0, a0);
}

// One entry of a frozen field of a kinematic run (rho, m, E): the update with R = 0.
// It changes nothing once the history is zero (which it is not where a run
// continues from another's checkpoint), so a steady AB2 step only reads the
// history; the stage sums and last stages of the other schemes add nothing.
constexpr int kFrozenFields = 5;
__host__ __device__ constexpr int frozen_field(int i) { return i < 4 ? i : 7; }
template <typename T>
__device__ __forceinline__ void frozen_entry(const UpdateArgs<T>& a, int mem, int i, int64_t idx) {
  const Update<T> up(a, mem, frozen_field(i));
  if (up.op == UP_RK_MID || up.op == UP_LAST) return;
  const cx<T> zero = mk<T>(0, 0), a0 = up.old_acc(idx);
  if (up.op == UP_AB2 && up.use_prev && a0.x == T(0) && a0.y == T(0)) return;
  up.apply(idx, zero, up.old_u(idx), a0);
}

// ------------------------------------------------------------------ k_zfwd_rhs
// Flat grid over (member, column tile of (ky, kx), output field), field fastest.
template <typename T, int N>
__global__ void __launch_bounds__((rhs_threads<T, N>()), (rhs_min_waves<T, N>())) k_zfwd_rhs(const RhsArgs<T> a) {
  using PL = PlanOf<N>;
  constexpr int C = rhs_tile<T, N>();
  constexpr int NT = rhs_threads<T, N>();
  constexpr int NH = Band<N>::NH, NHP = Band<N>::NHP, NBB = Band<N>::NB;
  constexpr int NCOLS = NBB * NHP;  // flattened (ky, kx) over the padded pitch
  using LP = LastPass<PL, C, NT>;
  __shared__ cx<T> tile[N * C];
  __shared__ cx<T> stw[N];
  const int tid = threadIdx.x;
  // fields 1..7 (or B alone); R_rho is formed by its own pass before this one,
  // because this pass overwrites m^ (which R_rho = -i k . m^ reads) with its next level
  const TileField tf = tile_field(a.nf);
  const int f = tf.field + a.f0;
  constexpr int ZT = (NCOLS + C - 1) / C;  // column tiles per member
  const int mem = tf.tile / ZT;
  const int c0 = (tf.tile - mem * ZT) * C;
  constexpr int64_t LS = NCOLS;             // plane stride of a compact spectrum (kz)
  constexpr int64_t LSZ = Pitch<T, N>::Z;  // plane stride of I_z (z)
  const int64_t ms = a.up.bt.mstride;
  const RhsMember<T> M(a, mem, f);

  // Output (i, r) of this thread's last-pass slots: compact index, or -1 for
  // a slot that is idle, a padding column or a dealiased kz.
  auto out_index = [&](int i, int r, int& kx, int& ky, int& kz) -> int64_t {
    int c, q;
    if (!last_slot<PL, C, NT, 0>(tid, i, r, c, q)) return -1;
    const int col = c0 + c;
    kx = col - (col / NHP) * NHP;
    if (col >= NCOLS || kx >= NH) return -1;
    ky = band_k<N>(col / NHP);
    const int l = pos_band<N>(q);
    if (l < 0) return -1;
    kz = band_k<N>(l);
    return (int64_t)l * LS + col;
  };
  // The state (for the update, and B^ for the resistive term) and the history
  cx<T> u_pre[LP::CNT][LP::R], r_pre[LP::CNT][LP::R];
  auto load_old = [&](int i, int r) {
    u_pre[i][r] = mk<T>(0, 0);
    r_pre[i][r] = mk<T>(0, 0);
    int kx, ky, kz;
    const int64_t idx = out_index(i, r, kx, ky, kz);
    if (idx < 0) return;
    u_pre[i][r] = M.up.old_u(idx);
    r_pre[i][r] = M.up.old_acc(idx);
  };
  auto load_all_old = [&] {
#pragma unroll
    for (int i = 0; i < LP::CNT; ++i)
#pragma unroll
      for (int r = 0; r < LP::R; ++r) load_old(i, r);
  };

  load_twiddles<T, PL, NT>(stw, a.tw, tid);
  cx<T> acc[LP::CNT][LP::R];
#pragma unroll
  for (int i = 0; i < LP::CNT; ++i)
#pragma unroll
    for (int r = 0; r < LP::R; ++r) acc[i][r] = mk<T>(0, 0);

  // Inputs of a flux group: value at (column c, position q)
  struct Group {
    const T *p0, *p1;
    T cf[2];
    int ax[2], nt;
  };
  auto group = [&](const OutSpec& sp) {
    Group G;
    G.nt = sp.nterms;
    G.p0 = member_ptr(a.flux[G.nt > 0 ? sp.t[0].src : 0], mem, ms);
    G.p1 = G.nt > 1 ? member_ptr(a.flux[sp.t[1].src], mem, ms) : G.p0;
    // the multipliers, converted once per group rather than once per element
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      G.cf[t] = t < G.nt ? T(sp.t[t].coef) : T(0);
      G.ax[t] = t < G.nt ? sp.t[t].axis : -1;
    }
    return G;
  };
  auto load = [&](const Group& G, int c, int q) -> cx<T> {
    const int col = c0 + c;
    cx<T> v = mk<T>(0, 0);
    const int kx = col - (col / NHP) * NHP;
    if (G.nt == 0 || col >= NCOLS || kx >= NH) return v;
    const int ky = band_k<N>(col / NHP);
    const int64_t idx = (int64_t)q * LSZ + col;
    const cx<T> x0 = ld(G.p0, idx);
    const cx<T> x1 = G.nt > 1 ? ld(G.p1, idx) : mk<T>(0, 0);
    const cx<T> xs[2] = {x0, x1};
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      if (t < G.nt) {
        if (G.ax[t] < 0) {
          v = cfma(G.cf[t], xs[t], v);
        } else {
          const T ck = G.cf[t] * T(G.ax[t] == 0 ? kx : ky);
          v = cfma(ck, ctimes_i(xs[t]), v);
        }
      }
    }
    return v;
  };
  auto add_A = [&](int i, int r, int, int, cx<T> v) { acc[i][r] = cadd(acc[i][r], v); };
  auto add_Z = [&](int i, int r, int, int q, cx<T> v) {  // + i kz v
    const int l = pos_band<N>(q);
    const T kz = T(l < 0 ? 0 : band_k<N>(l));
    acc[i][r] = cfma(kz, ctimes_i(v), acc[i][r]);
  };
  if constexpr (rhs_upfront<N>()) {
    const Group GA = group(a.A[f]), GZ = group(a.Z[f]);
    using FP = FirstPass<PL, C, NT>;
    cx<T> x[FP::CNT][FP::R], z[FP::CNT][FP::R];
    auto load_all = [&](const Group& G, cx<T> (&w)[FP::CNT][FP::R]) {
#pragma unroll
      for (int i = 0; i < FP::CNT; ++i) {
        int c, j;
        const bool ok = first_slot<C, FP::NBF, NT, 0>(tid, i, c, j);
#pragma unroll
        for (int r = 0; r < FP::R; ++r) w[i][r] = ok ? load(G, c, j + r * FP::NBF) : mk<T>(0, 0);
      }
    };
    load_all(GA, x);
    load_all(GZ, z);
    __syncthreads();  // the twiddles
    if (GA.nt > 0) {  // uniform across the block
      fft_first_regs<T, PL, C, NT, C, 1, -1, 0, 0>(tile, x, tid, C, add_A);
      fft_rest<T, PL, C, NT, C, 1, -1, 0, 0>(tile, stw, tid, C, add_A);
    }
    if (GZ.nt > 0) {
      __syncthreads();  // the LDS tile is about to be rewritten
      fft_first_regs<T, PL, C, NT, C, 1, -1, 0, 0>(tile, z, tid, C, add_Z);
      fft_rest<T, PL, C, NT, C, 1, -1, 0, 0>(tile, stw, tid, C, add_Z);
    }
  } else if constexpr (N <= 96) {
    // one code for both groups, where the launch is short enough for its instruction
    // fetch to show (64 FP32: 17.8 us written out, 16.2 as a loop)
#pragma unroll 1
    for (int grp = 0; grp < 2; ++grp) {
      const Group G = group(grp == 0 ? a.A[f] : a.Z[f]);
      if (G.nt == 0) continue;
      if (grp == 1) __syncthreads();
      fft_reg<T, PL, C, NT, C, 1, -1>(tile, stw, tid, C, [&](int c, int q) { return load(G, c, q); },
                                      [&](int i, int r, int c, int q, cx<T> v) {
                                        if (grp == 0) add_A(i, r, c, q, v);
                                        else add_Z(i, r, c, q, v);
                                      });
    }
  } else {
    // written out, which takes fewer registers (256 FP32 70 -> 63: 224 -> 213 us)
    const Group GA = group(a.A[f]), GZ = group(a.Z[f]);
    if (GA.nt > 0)
      fft_reg<T, PL, C, NT, C, 1, -1>(tile, stw, tid, C, [&](int c, int q) { return load(GA, c, q); }, add_A);
    if (GZ.nt > 0) {
      if (GA.nt > 0) __syncthreads();
      fft_reg<T, PL, C, NT, C, 1, -1>(tile, stw, tid, C, [&](int c, int q) { return load(GZ, c, q); }, add_Z);
    }
  }
  // epilogue over this thread's last-pass positions; all its loads go out
  // together, ahead of the first that is used
  load_all_old();
#pragma unroll
  for (int i = 0; i < LP::CNT; ++i) {
#pragma unroll
    for (int r = 0; r < LP::R; ++r) {
      int kx, ky, kz;
      const int64_t idx = out_index(i, r, kx, ky, kz);
      if (idx < 0) continue;
      M.template apply<(N >= 512)>(idx, acc[i][r], u_pre[i][r], r_pre[i][r], kx, ky, kz);
    }
  }
}

// ------------------------------------------------------------------ k_row
// blockIdx.x = row pair p: rows (z, 2y') and (z, 2y'+1), z = p / (N/2).
template <int MODE> struct RowShape;
template <> struct RowShape<RM_XA> { static constexpr int NIN = 4, NOUT = 3, NB = 4; };
template <> struct RowShape<RM_XB> { static constexpr int NIN = 16, NOUT = 12, NB = 16; };
template <> struct RowShape<RM_XL> { static constexpr int NIN = 11, NOUT = 12, NB = 12; };
template <> struct RowShape<RM_XFWD_REAL> { static constexpr int NIN = 8, NOUT = 8, NB = 8; };
template <> struct RowShape<RM_XINV_REAL> { static constexpr int NIN = 8, NOUT = 8, NB = 8; };
template <> struct RowShape<RM_XFWD_ONE> { static constexpr int NIN = 1, NOUT = 1, NB = 1; };
template <> struct RowShape<RM_XINV_ONE> { static constexpr int NIN = 1, NOUT = 1, NB = 1; };
template <> struct RowShape<RM_XK> { static constexpr int NIN = 8, NOUT = 3, NB = 8; };
template <> struct RowShape<RM_XDIAG> { static constexpr int NIN = kDiagFields, NOUT = 0, NB = kDiagFields; };

template <typename T>
__device__ __forceinline__ bool finite_(T v) { return isfinite(v); }

// 1/x and sqrt(x) of the pointwise stages.  FP32: the hardware v_rcp_f32 and
// v_sqrt_f32 (1 ulp) instead of the correctly rounded sequences (about ten
// instructions each), in the VALU-bound flux and velocity passes; the
// difference is at the level of FP32 rounding.  FP64: correctly rounded.
template <typename T> __device__ __forceinline__ T recip_(T x) { return T(1) / x; }
template <> __device__ __forceinline__ float recip_<float>(float x) { return __builtin_amdgcn_rcpf(x); }
template <typename T> __device__ __forceinline__ T sqrt_(T x) { return sqrt(x); }
template <> __device__ __forceinline__ float sqrt_<float>(float x) { return __builtin_amdgcn_sqrtf(x); }

// Fixed-order tree reduction over the block (sum, or NaN-propagating max);
// the result is valid in thread 0.  Deterministic for a given launch shape.
template <int NT = kThreads>
__device__ __forceinline__ double block_reduce(double v, bool is_max, double* s, int tid) {
  __syncthreads();
  s[tid] = v;
  __syncthreads();
  for (int w = NT / 2; w > 0; w >>= 1) {
    if (tid < w) {
      const double o = s[tid + w];
      if (is_max) {
        if (!(o <= s[tid])) s[tid] = o;
      } else {
        s[tid] += o;
      }
    }
    __syncthreads();
  }
  return s[0];
}

// Error-free sum of s and x (Neumaier's two-sum): s <- fl(s + x), the
// rounding error of that addition added to the compensation c.
__device__ __forceinline__ void neumaier_add(double& s, double& c, double x) {
  const double t = s + x;
  if (fabs(s) >= fabs(x)) c += (s - t) + x;
  else c += (x - t) + s;
  s = t;
}

// Compensated fixed-order tree sum over the block of per-thread (sum,
// compensation) pairs; every level adds with neumaier_add, so the block
// result carries the same compensation as a serial Neumaier sum.  s: 2 NT
// doubles of LDS scratch.  The result (s + c) is valid in thread 0.
template <int NT = kThreads>
__device__ __forceinline__ double block_sum_comp(double v, double cv, double* s, int tid) {
  __syncthreads();
  s[tid] = v;
  s[NT + tid] = cv;
  __syncthreads();
  for (int w = NT / 2; w > 0; w >>= 1) {
    if (tid < w) {
      double a = s[tid], ca = s[NT + tid] + s[NT + tid + w];
      neumaier_add(a, ca, s[tid + w]);
      s[tid] = a;
      s[NT + tid] = ca;
    }
    __syncthreads();
  }
  return s[0] + s[NT];
}

// Persistent: workgroup w handles row pairs w, w + G, w + 2G, ... (G = grid
// size, sized by the host to the number of resident workgroups).  For the
// spectral-input modes the global loads of the next row pair's first FFT pass
// are issued right after the current pair's first pass, so they are in flight
// during the current pair's LDS passes, pointwise work and stores.
// Fold a workgroup's CFL speed and non-finite count into its own status slot
// of a member (slot = workgroup id; kStatusSlots slots of two doubles: the
// largest signal speed seen by any step since the state was set, and the
// count of non-finite points).  The speed is reduced in FP64 (a max, exact in
// any precision, NaN propagating) and kept as a running max over steps; each
// slot has a single writer, so no atomics are needed and the result does not
// depend on workgroup order.  Block-uniform call.  s_red: NT doubles of LDS
// scratch, which may alias the caller's row buffer (the reductions begin and
// end with a barrier).
template <int NT>
__device__ __forceinline__ void flush_status(double cfl, int bad, double* slots, double* s_red) {
  const int tid = threadIdx.x;
  const double cfl_b = block_reduce<NT>(cfl, true, s_red, tid);
  const double bad_b = block_reduce<NT>(double(bad), false, s_red, tid);
  __syncthreads();  // every thread has read the results before the scratch is reused
  if (tid == 0) {
    double* const slot = slots + 2 * (int64_t)blockIdx.x;
    const double old = slot[0];
    slot[0] = !(cfl_b <= old) ? cfl_b : old;
    slot[1] = slot[1] + bad_b;
  }
}

// Threads of a row pass: FP32 rows of N >= 1024 take 512, which keeps the
// per-thread first-pass work (and registers) of N = 512 on 256 threads.  The
// FP32 flux pass at N = 512, 384 and 256 also takes 512: with wave maps each
// wave then owns two fields instead of four, the registers fit 128, and its LDS
// tile still allows two workgroups per CU, so four waves per SIMD run instead
// of two (13% faster at 512) or three (3% at 256).  The FP32 velocity pass at
// N = 256 takes 128: two waves of two fields each, whose 32-butterfly radix-8
// passes then fill every lane (256 threads left half of them idle; 19%).
// The FP64 velocity pass at 256 takes 128 as well (252 -> 173 us), and so do 96 (FP64
// 18.9 -> 16.9), FP32 at 192 (55.3 -> 53.5) and at 512 (655 -> 629); FP32 at 384 takes
// one wave (348 -> 324).
// The FP64 flux pass at N = 512, 384 and 192 takes 512 too (at 512 one workgroup
// per CU: two waves per SIMD instead of one, 6.78 -> 5.63 ms; 192 324 -> 307 us).
// Below 256 (wave maps at 64 and 128): the velocity pass takes one wave per row
// pair, which then needs no barrier (64: 11.1 -> 9.1 us FP64; 128: 36.6 ->
// 32.4 us FP64, 22.6 -> 20.3 us FP32), the flux pass as many threads as let
// every lane of a first pass hold a butterfly (128: 256 threads in FP32, 56.8 ->
// 55.1 us) or half as many (64, and 128 in FP64 where the registers of two
// butterflies fit: 20.2 -> 18.5 and 109 -> 89 us; FP32 at 128 would spill).
// The passes from and to real fields take a thread per first-pass butterfly at 384
// and 512 (set_state at 512 FP32 4.15 -> 3.39 ms, FP64 10.55 -> 7.89), and so does the
// one to real fields at 768, whose three butterflies per thread at 256 threads could not
// be paired (first_slot map 2: no mirror is read again; get_state 13.0 -> 12.0 ms mixed;
// the one from real fields loses there, 11.1 -> 11.5).
// The kinematic pass (eight fields) does the same.
// The flux passes of a full run: RM_XL leaves out the strains (the Laplacian viscous
// force of a run is added spectrally).
constexpr bool is_flux(int mode) { return mode == RM_XB || mode == RM_XL; }
// The passes from and to real fields of a call on one field (mhd_fft3d, the gradient
// of mhd_spectra) take one wave and one field's LDS per row pair: in the eight-field
// passes' workgroups seven of eight threads have nothing to do (mhd_fft3d in those ->
// in these: 512 FP32 forward 420 -> 405 us, inverse 581 -> 412; 384 FP32 258 -> 181 and
// 264 -> 187; 192 FP64 56 -> 41 and 63 -> 47; up to 64 within the launch time).
constexpr bool from_real(int mode) { return mode == RM_XFWD_REAL || mode == RM_XFWD_ONE; }
constexpr bool to_real(int mode) { return mode == RM_XINV_REAL || mode == RM_XINV_ONE; }
template <typename T, int N, int MODE> constexpr int row_threads() {
  if (MODE == RM_XFWD_ONE || MODE == RM_XINV_ONE) return 64;
  if (MODE == RM_XK) {
    constexpr int w = 8 * (N / PlanOf<N>::r[0]);
    return w <= 64 ? 64 : (w >= 512 ? 512 : (w + 63) / 64 * 64);
  }
  if (is_flux(MODE) && (N == 512 || N == 384 || (sizeof(T) == 4 && N == 256))) return 2 * kThreads;
  if (is_flux(MODE) && (N == 64 || (sizeof(T) == 8 && N == 128))) return kThreads / 2;
  if (is_flux(MODE) && sizeof(T) == 8 && N == 192) return 2 * kThreads;
  if (MODE == RM_XA && (N == 64 || N == 128 || (N == 192 && sizeof(T) == 8) || (N == 384 && sizeof(T) == 4))) return 64;
  if (MODE == RM_XA && (N == 96 || N == 192 || N == 256 || (N == 512 && sizeof(T) == 4))) return kThreads / 2;
  if ((MODE == RM_XFWD_REAL || MODE == RM_XINV_REAL) && (N == 384 || N == 512)) return 2 * kThreads;
  if (MODE == RM_XINV_REAL && N == 768) return 2 * kThreads;
  return (sizeof(T) == 4 && N >= 1024) ? 2 * kThreads : kThreads;
}

// Register caps of the FP32 row passes: two waves per SIMD from N = 256 on (the
// 512-thread flux passes come out at 128 registers or fewer, four waves per SIMD,
// which is what their LDS allows).  Left free, a flux pass can take more than 256
// registers and then runs one wave per SIMD.
template <typename T, int N, int MODE> constexpr int row_min_blocks() {
  if (sizeof(T) != 4 || row_threads<T, N, MODE>() < kThreads || MODE == RM_XK) return 1;
  if (is_flux(MODE) && (N == 512 || N == 384 || N == 256)) return 2;
  return 2 * kThreads / row_threads<T, N, MODE>();
}

template <typename T, int N, int MODE>
__global__ void __launch_bounds__((row_threads<T, N, MODE>()), (row_min_blocks<T, N, MODE>()))
    k_row(const RowArgs<T> a) {
  using PL = PlanOf<N>;
  constexpr int NT = row_threads<T, N, MODE>();
  constexpr int K = Band<N>::K, PY = Pitch<T, N>::Y;
  constexpr int NH = Band<N>::NH;
  constexpr int NB = RowShape<MODE>::NB;
  // LDS row layout, chosen per pass by measurement.  Linear addressing where
  // the precomputed addresses would push a pass past 256 registers into
  // spills (the flux pass at N = 1024, the diagnostics pass from 768: 308 bytes of
  // scratch there, 16.2 ms; linear 219 registers at 512 threads, 238 at 256, and
  // diagnostics of 17.8 and 15.7 ms instead of 25.4).  The stage swizzle
  // (conflict-free LDS access, but more address arithmetic) where it measured
  // faster: the flux pass below N = 512 (3%) and the velocity pass from N = 512
  // (2%).  Otherwise one padding slot per 8 elements.
  constexpr bool LIN = (is_flux(MODE) && N >= 1024) || (MODE == RM_XDIAG && N >= 768);
  constexpr bool SWZ = !LIN && N % 16 == 0 && N >= 128 && ((is_flux(MODE) && N < 512) || (MODE == RM_XA && N >= 512));
  constexpr int PADSH = 3;
  constexpr int LAY = SWZ ? kSwizzle : (PADSH | (LIN ? kLinear : 0));
  // row pitch in LDS: swizzled rows are shifted by 16 elements from row to
  // row, so that a 32-lane read spanning two rows of N = 128 uses all banks
  constexpr int BS = SWZ ? N + 16 : N + (N >> PADSH) + 1;
  constexpr bool SPEC_IN = !from_real(MODE);
  // Wave maps: each field's transforms stay inside one wave, so a wave-level
  // fence replaces the workgroup barrier between passes and only the
  // pointwise stage, which reads every field at one point, is bracketed by
  // barriers.  Used (measured) by the velocity and flux passes from N = 384
  // (12% and 5% faster at 512), at 256, 128 and 64 (with the thread counts of
  // row_threads) and by the one-wave FP64 velocity pass at 192 (94 -> 85 us); not
  // at 96 and 192 otherwise (their 12 and 32 first-pass butterflies per field
  // leave lanes of a wave idle: 96 FP32 flux pass 30.8 -> 35.7 us) or with fewer
  // fields than waves.
  constexpr bool FLUX = is_flux(MODE) || MODE == RM_XK;  // forms fluxes and the status
  constexpr bool WAVE = MODE == RM_XK ? is_pow2(N) && N >= 64
                                      : (MODE == RM_XA || is_flux(MODE)) &&
                                            (N >= 384 || N == 256 || N == 128 || N == 64 || (N == 192 && NT == 64)) &&
                                            NB >= NT / 64;
  constexpr int RMAP = WAVE ? 3 : 1;
  using FP = FirstPass<PL, NB, NT, RMAP>;
  auto at = [](int b, int pos) { return lds_at<1, BS, LAY, PL, 0>(b, pos); };
  __shared__ cx<T> buf[NB * BS];
  __shared__ cx<T> stw[N];
  // block reductions (status words, diagnostics) use the row buffer as scratch
  // when it is large enough (each begins with a barrier, after which no row
  // work touches the buffer); small sizes get their own array
  constexpr bool RED_IN_BUF = sizeof(cx<T>) * NB * BS >= 2 * NT * sizeof(double);
  __shared__ double red_own[RED_IN_BUF ? 1 : 2 * NT];
  double* const red = RED_IN_BUF ? reinterpret_cast<double*>(buf) : red_own;
  const int tid = threadIdx.x;
  const int64_t rows_per_mem = (int64_t)N * N / 2;
  const int64_t nitems = rows_per_mem * a.bt.nmem;
  const int nin = (MODE == RM_XFWD_REAL || MODE == RM_XINV_REAL) ? a.nf : RowShape<MODE>::NIN;
  const int nout = (MODE == RM_XFWD_REAL || MODE == RM_XINV_REAL)
                       ? a.nf
                       : ((MODE == RM_XA && a.nf == 4) ? 4 : RowShape<MODE>::NOUT);
  load_twiddles<T, PL, NT>(stw, a.tw, tid);
  // with wave maps no workgroup barrier comes before the first pass that reads
  // the twiddles, which other waves loaded
  if constexpr (WAVE) __syncthreads();
  auto lds_store = [&](int, int, int fld, int q, cx<T> v) { buf[at(fld, q)] = v; };

  // Prefetch registers for the next row pair: the two rows' Hermitian
  // half-spectrum entries X0[q], X1[q] behind the first-pass elements in the
  // lower half (q < N/2, r < R/2).  Elements q >= N-K use X[N-q]: with paired
  // first-pass slots (FMAP 2) that is a lower-half element of the thread's
  // partner butterfly, already in these registers; with FMAP 3 it is in a
  // partner lane's registers; otherwise (FMAP 1) a mirror lane prefetched it
  // and it is read again when used.
  // FMAP 3: plain slots, but when NBF divides the wave width the partner
  // butterfly NBF - j sits in the same wave and the mirror comes by a lane
  // shuffle of its register.
  constexpr int RH = FP::R / 2;
  constexpr int FMAP = (FP::CNT % 2 == 0 && FP::NBF % 2 == 0) ? 2 : ((FP::NBF >= 2 && 64 % FP::NBF == 0) ? 3 : 1);
  constexpr int HC = FP::CNT / 2;
  constexpr int FM1 = !SPEC_IN ? 1 : (FMAP == 2 ? (WAVE ? 4 : 2) : RMAP);  // lane map of the first pass
  // first-pass rows r whose positions j + r NBF all lie in the dealiased gap:
  // known zeros, neither loaded nor assembled, and pruned from the DFT
  constexpr unsigned ZROWS = gap_rows<N, FP::NBF, FP::R, K>();
  cx<T> p0[FP::CNT][RH], p1[FP::CNT][RH];
  auto issue = [&](int64_t item) {
    const int mi = (int)(item / rows_per_mem);
    const int64_t row0 = 2 * (item - mi * rows_per_mem);
    const T* in0 = member_ptr(a.in0, mi, a.bt.mstride);
#pragma unroll
    for (int i = 0; i < FP::CNT; ++i) {
      int b, j;
      const bool ok = first_slot<NB, FP::NBF, NT, FM1>(tid, i, b, j) && b < nin;
      const T* src = in0 + 2 * b * a.in_stride;
#pragma unroll
      for (int r = 0; r < RH; ++r) {
        const int q = j + r * FP::NBF;
        p0[i][r] = mk<T>(0, 0);  // the previous pair's values are dead
        p1[i][r] = mk<T>(0, 0);
        if ((ZROWS >> r) & 1u) continue;
        if (ok && q <= K) {
          p0[i][r] = ld(src, row0 * PY + q);
          p1[i][r] = ld(src, (row0 + 1) * PY + q);
        }
      }
    }
  };
  // Real rows, as row0 + i row1.  From N = 96 the next pair's are prefetched into the
  // first-pass elements too (loaded, transformed and stored in turn the pass waits on
  // memory three quarters of its time: set_state at 512 FP64 7.9 -> 6.4 ms, 384 FP32
  // 1.49 -> 1.39; 192 178 -> 172 us); smaller ones go to the LDS, a point per thread
  // (few of the threads hold a butterfly there), and so do FP64 rows of an FP32 run up to
  // 128, whose conversion waits for the load and so undoes the prefetch (RUNTIME:
  // set_state from FP64 at 128 prefetched 58.2, so 55.0 us; at 96 31.0 and 29.9; kept
  // unconverted instead, twice the registers, 56.4 and 30.5, and FP32 rows slower).
  constexpr bool REAL_REGS = !SPEC_IN && N >= 96;
  constexpr bool RUNTIME = REAL_REGS && sizeof(T) == 4 && N <= 128;
  const bool real_regs = REAL_REGS && !(RUNTIME && a.real_dtype == 0);
  auto real_pair = [&](auto* in, int64_t e) { return mk<T>(T(in[e]), T(in[e + N])); };
  cx<T> rx[REAL_REGS ? FP::CNT : 1][FP::R];
  auto issue_real = [&](int64_t item) {
    auto rows = [&](auto* in) {
#pragma unroll
      for (int i = 0; i < FP::CNT; ++i) {
        int b, j;
        const bool ok = first_slot<NB, FP::NBF, NT, FM1>(tid, i, b, j) && b < nin;
#pragma unroll
        for (int r = 0; r < FP::R; ++r)
          rx[i][r] = ok ? real_pair(in, b * a.g.n3 + 2 * item * N + j + r * FP::NBF) : mk<T>(0, 0);
      }
    };
    if (a.real_dtype == 0) rows(static_cast<const double*>(a.real_in));
    else rows(static_cast<const float*>(a.real_in));
  };
  // per-workgroup accumulators of the diagnostic / status modes: the largest
  // signal speed (each point's speed is formed in T, and the thread's maximum
  // of T values is exact in T; it goes to FP64 at the workgroup's flush) and
  // the non-finite count of the flux pass; Neumaier (sum, compensation) pairs
  // of the diagnostics pass
  T cfl = T(0);
  int bad = 0;
  double q[kDiagQ], qc[kDiagQ];
#pragma unroll
  for (int i = 0; i < kDiagQ; ++i) {
    q[i] = 0.0;
    qc[i] = 0.0;
  }

  int64_t item = blockIdx.x;
  if constexpr (SPEC_IN) {
    if (item < nitems) issue(item);
  } else if constexpr (REAL_REGS) {
    if (real_regs && item < nitems) issue_real(item);
  }
  int cur_m = -1;  // member whose CFL / non-finite status is being accumulated
  for (; item < nitems; item += gridDim.x) {
    const int mem = (int)(item / rows_per_mem);
    const int64_t row0 = 2 * (item - mem * rows_per_mem);  // flattened row z*N + y of the first row
    if constexpr (FLUX) {
      if (mem != cur_m) {  // uniform across the workgroup
        if (cur_m >= 0 && a.status) {
          flush_status<NT>(double(cfl), bad, member_ptr(a.status, cur_m, a.bt.mstride), red);
          cfl = T(0);
          bad = 0;
        }
        cur_m = mem;
      }
    }
    // the previous row pair is done with the LDS (with wave maps a wave only
    // writes its own fields before the next barrier, and it is the only one
    // that still reads them)
    if constexpr (!WAVE) __syncthreads();
    if constexpr (!SPEC_IN) {
      if (real_regs) {
        if constexpr (REAL_REGS) {
          fft_first_regs<T, PL, NB, NT, 1, BS, -1, FM1, LAY>(buf, rx, tid, nin, lds_store);
          if (item + gridDim.x < nitems) issue_real(item + gridDim.x);
        }
      } else {
        for (int e = tid; e < nin * N; e += NT) {
          const int fld = e / N, x = e - (e / N) * N;
          const int64_t base = fld * a.g.n3 + row0 * N + x;
          buf[at(fld, x)] = a.real_dtype == 0 ? real_pair(static_cast<const double*>(a.real_in), base)
                                              : real_pair(static_cast<const float*>(a.real_in), base);
        }
        if constexpr (RUNTIME) {
          __syncthreads();
          fft_pass_valu<T, PL, NB, NT, 1, BS, -1, 0, RMAP, LAY>(buf, stw, tid, nin);
        }
      }
    } else {
      // inverse x transform: first pass from the prefetched registers
      // first-pass inputs Z[q] = X0[q] + i X1[q] (q <= K),
      // Z[N-k] = conj(X0[k]) + i conj(X1[k]) (k <= K), zero in the gap.
      // Rows r < R/2 hold q < N/2, rows r >= R/2 hold q > N/2 (mirrors of
      // q < N/2).  The prefetch registers are zero wherever nothing was loaded
      // (q > K, or an idle slot), so both formulas give zero in the gap with no
      // case analysis.  (At q = 0 the formula also adds the imaginary parts of
      // the two rows' DC terms, which are zero up to rounding.)
      cx<T> v[FP::CNT][FP::R];
#pragma unroll
      for (int i = 0; i < FP::CNT; ++i) {
        int b, j;
        const bool ok = first_slot<NB, FP::NBF, NT, FM1>(tid, i, b, j) && b < nin;
        const T* src = member_ptr(a.in0, mem, a.bt.mstride) + 2 * b * a.in_stride;
        // FMAP 3: lane of butterfly NBF - j (j = tid mod NBF since NBF divides 64)
        const int plane = (tid & 63) - j + (FP::NBF - j) % FP::NBF;
#pragma unroll
        for (int r = 0; r < FP::R; ++r) {
          if ((ZROWS >> r) & 1u) {
            v[i][r] = mk<T>(0, 0);
            continue;
          }
          if (r < RH) {
            const cx<T> x0 = p0[i][r < RH ? r : 0], x1 = p1[i][r < RH ? r : 0];
            v[i][r] = mk<T>(x0.x - x1.y, x0.y + x1.x);
            continue;
          }
          // mirror element X[N - q]: element R-r-1 of butterfly NBF-j, or, for
          // j = 0, element R-r of the same butterfly (none for r = R/2: that is
          // q = N/2, in the gap)
          const int r1 = (FP::R - 1 - r) < RH ? (FP::R - 1 - r) : 0;
          const bool self_ok = (FP::R - r) < RH;
          const int r0 = self_ok ? (FP::R - r) : 0;
          const cx<T> zero = mk<T>(0, 0);
          const cx<T> self0 = self_ok ? p0[i][r0] : zero, self1 = self_ok ? p1[i][r0] : zero;
          cx<T> x0 = zero, x1 = zero;
          if constexpr (FMAP == 3) {
            // uniform: every lane takes part in the shuffles
            const cx<T> s0 = mk<T>(__shfl(p0[i][r1].x, plane), __shfl(p0[i][r1].y, plane));
            const cx<T> s1 = mk<T>(__shfl(p1[i][r1].x, plane), __shfl(p1[i][r1].y, plane));
            x0 = j == 0 ? self0 : s0;
            x1 = j == 0 ? self1 : s1;
          } else if constexpr (FMAP == 2) {
            // the partner butterfly is the partner slot, except j = 0 (see
            // above) and j = NBF/2, its own partner
            const int ip = i < HC ? i + HC : i - HC;
            if (j == 0) {
              x0 = self0;
              x1 = self1;
            } else if (j == FP::NBF / 2) {
              x0 = p0[i][r1];
              x1 = p1[i][r1];
            } else {
              x0 = p0[ip][r1];
              x1 = p1[ip][r1];
            }
          } else {
            const int q = j + r * FP::NBF;
            if (ok && q >= N - K) {
              x0 = ld(src, row0 * PY + (N - q));
              x1 = ld(src, (row0 + 1) * PY + (N - q));
            }
          }
          v[i][r] = mk<T>(x0.x + x1.y, x1.x - x0.y);
        }
      }
      fft_first_regs<T, PL, NB, NT, 1, BS, +1, FM1, LAY, ZROWS>(buf, v, tid, nin, lds_store);
      if (item + gridDim.x < nitems) issue(item + gridDim.x);  // next pair's loads overlap the rest
      fft_rest<T, PL, NB, NT, 1, BS, +1, RMAP, LAY, true>(buf, stw, tid, nin, lds_store);
    }
    if constexpr (!REAL_REGS) __syncthreads();

    if constexpr (to_real(MODE)) {
      for (int e = tid; e < nout * N; e += NT) {
        const int fld = e / N, x = e - (e / N) * N;
        const cx<T> z = buf[at(fld, x)];
        const int64_t base = fld * a.g.n3 + row0 * N + x;
        if (a.real_dtype == 0) {
          static_cast<double*>(a.real_out)[base] = double(z.x);
          static_cast<double*>(a.real_out)[base + N] = double(z.y);
        } else {
          static_cast<float*>(a.real_out)[base] = float(z.x);
          static_cast<float*>(a.real_out)[base + N] = float(z.y);
        }
      }
      continue;
    }

    if constexpr (MODE == RM_XA) {
      // u = m / rho, both rows at once; with four outputs also q = |u|^2/2
      // (the viscous-force variant's energy term) into the slot m_z vacated
      for (int x = tid; x < N; x += NT) {
        const cx<T> rho = buf[at(0, x)];
        const T i0 = recip_(rho.x), i1 = recip_(rho.y);
        cx<T> u[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
          const cx<T> m = buf[at(1 + i, x)];
          u[i] = mk<T>(m.x * i0, m.y * i1);
          buf[at(i, x)] = u[i];
        }
        if (nout == 4)
          buf[at(3, x)] = mk<T>(T(0.5) * (u[0].x * u[0].x + u[1].x * u[1].x + u[2].x * u[2].x),
                                T(0.5) * (u[0].y * u[0].y + u[1].y * u[1].y + u[2].y * u[2].y));
      }
    }

    if constexpr (is_flux(MODE)) {
      // Real-space fluxes of Eqs. MHD2-MHD4 at every point of both rows.
      // Inputs: 0 rho, 1-3 m, 4-6 B, 7 E, 8 S_xx, 9 S_yy, 10 S_xy, 11 S_xz,
      // 12 S_yz, 13-15 J (RM_XL: 8-10 J).  Outputs: 0 Pi_xx, 1 Pi_yy, 2 Pi_zz, 3 Pi_xy,
      // 4 Pi_xz, 5 Pi_yz, 6-8 F^E, 9-11 e = u x B.
      const T gm1 = T(a.gamma[mem] - 1.0), gam = T(a.gamma[mem]), two_nu = T(2.0 * a.nu[mem]),
              eta = T(a.eta[mem]);
      constexpr bool STRAIN = MODE == RM_XB;
      constexpr int NV = RowShape<MODE>::NIN;
      auto point = [&](const T (&v)[NV], T (&out)[12]) {
        const T rho = v[0], mx = v[1], my = v[2], mz = v[3];
        const T Bx = v[4], By = v[5], Bz = v[6], E = v[7];
        const T Jx = v[NV - 3], Jy = v[NV - 2], Jz = v[NV - 1];
        const T ir = recip_(rho);
        const T ux = mx * ir, uy = my * ir, uz = mz * ir;
        const T B2 = Bx * Bx + By * By + Bz * Bz;
        const T P = gm1 * (E - T(0.5) * (mx * ux + my * uy + mz * uz) - T(0.5) * B2);
        const T Pt = P + T(0.5) * B2;
        out[0] = mx * ux + Pt - Bx * Bx;
        out[1] = my * uy + Pt - By * By;
        out[2] = mz * uz + Pt - Bz * Bz;
        out[3] = mx * uy - Bx * By;
        out[4] = mx * uz - Bx * Bz;
        out[5] = my * uz - By * Bz;
        const T uB = ux * Bx + uy * By + uz * Bz;
        const T EP = E + Pt;
        out[6] = EP * ux - uB * Bx;
        out[7] = EP * uy - uB * By;
        out[8] = EP * uz - uB * Bz;
        if constexpr (STRAIN) {
          const T Sxx = v[8], Syy = v[9], Sxy = v[10], Sxz = v[11], Syz = v[12];
          const T Szz = -(Sxx + Syy);
          const T vr = two_nu * rho;
          out[0] -= vr * Sxx;
          out[1] -= vr * Syy;
          out[2] -= vr * Szz;
          out[3] -= vr * Sxy;
          out[4] -= vr * Sxz;
          out[5] -= vr * Syz;
          out[6] -= vr * (ux * Sxx + uy * Sxy + uz * Sxz);
          out[7] -= vr * (ux * Sxy + uy * Syy + uz * Syz);
          out[8] -= vr * (ux * Sxz + uy * Syz + uz * Szz);
        }
        out[6] -= eta * (By * Jz - Bz * Jy);
        out[7] -= eta * (Bz * Jx - Bx * Jz);
        out[8] -= eta * (Bx * Jy - By * Jx);
        out[9] = uy * Bz - uz * By;
        out[10] = uz * Bx - ux * Bz;
        out[11] = ux * By - uy * Bx;
        // fastest signal speed for the CFL limit, and a non-finite check
        const T umax = fmax(fabs(ux), fmax(fabs(uy), fabs(uz)));
        const T c = umax + sqrt_((gam * P + B2) * ir);
        if (!(c <= cfl)) cfl = c;  // NaN propagates
        const bool fin = finite_(rho) && finite_(mx) && finite_(my) && finite_(mz) && finite_(Bx) &&
                         finite_(By) && finite_(Bz) && finite_(E);
        bad += fin ? 0 : 1;
      };
      // FP64 rows too short to give every thread a point of both rows: a thread
      // takes a point of one row (half the serial work and registers per
      // thread: flux pass at 96 56 -> 48 us, at 64 20.2 -> 19.1 us).  In FP32 the
      // narrower LDS accesses cost as much as that saves (256: 360 -> 371 us).
      constexpr bool HSPLIT = sizeof(T) == 8 && (2 * N + NT - 1) / NT < 2 * ((N + NT - 1) / NT);
      if constexpr (HSPLIT) {
        T* const bt = reinterpret_cast<T*>(buf);
        for (int e = tid; e < 2 * N; e += NT) {
          const int h = e >= N ? 1 : 0, x = e - h * N;
          T v[NV], o[12];
#pragma unroll
          for (int f = 0; f < NV; ++f) v[f] = bt[2 * at(f, x) + h];
          point(v, o);
#pragma unroll
          for (int k = 0; k < 12; ++k) bt[2 * at(k, x) + h] = o[k];
        }
      } else {
        for (int x = tid; x < N; x += NT) {
          cx<T> v[NV], o[12];
#pragma unroll
          for (int f = 0; f < NV; ++f) v[f] = buf[at(f, x)];
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            T vh[NV], oh[12];
#pragma unroll
            for (int f = 0; f < NV; ++f) vh[f] = h == 0 ? v[f].x : v[f].y;
            point(vh, oh);
#pragma unroll
            for (int k = 0; k < 12; ++k) {
              if (h == 0) o[k].x = oh[k];
              else o[k].y = oh[k];
            }
          }
#pragma unroll
          for (int k = 0; k < 12; ++k) buf[at(k, x)] = o[k];
        }
      }
    }

    if constexpr (MODE == RM_XDIAG) {
      // Inputs: 0 rho, 1-3 m, 4-6 B, 7 E, 8 div B.  (The current's mean square is
      // a spectral sum, exact by Parseval for the band-limited B^.)
      const double gm1 = a.gamma[mem] - 1.0, gam = a.gamma[mem];
      for (int x = tid; x < N; x += NT) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          auto g = [&](int f) -> double { const cx<T> v = buf[at(f, x)]; return double(h == 0 ? v.x : v.y); };
          const double rho = g(0), mx = g(1), my = g(2), mz = g(3), Bx = g(4), By = g(5), Bz = g(6), E = g(7);
          const double dB = g(8);
          const double ux = mx / rho, uy = my / rho, uz = mz / rho;
          const double B2 = Bx * Bx + By * By + Bz * Bz;
          const double mu = mx * ux + my * uy + mz * uz;
          const double P = gm1 * (E - 0.5 * mu - 0.5 * B2);
          auto acc = [&](int i, double x) { neumaier_add(q[i], qc[i], x); };
          acc(DQ_RHO, rho);
          acc(DQ_MX, mx);
          acc(DQ_MY, my);
          acc(DQ_MZ, mz);
          acc(DQ_EKIN, 0.5 * mu);
          acc(DQ_EMAG, 0.5 * B2);
          acc(DQ_P, P);
          acc(DQ_E, E);
          acc(DQ_HC, ux * Bx + uy * By + uz * Bz);
          acc(DQ_UABS, sqrt(ux * ux + uy * uy + uz * uz));
          acc(DQ_BABS, sqrt(B2));
          const double adb = fabs(dB);
          if (!(adb <= q[DQ_DIVB_MAX])) q[DQ_DIVB_MAX] = adb;
          const double c = fmax(fabs(ux), fmax(fabs(uy), fabs(uz))) + sqrt((gam * P + B2) / rho);
          if (!(c <= q[DQ_CFL_MAX])) q[DQ_CFL_MAX] = c;
          const bool fin = isfinite(rho) && isfinite(mx) && isfinite(my) && isfinite(mz) && isfinite(Bx) &&
                           isfinite(By) && isfinite(Bz) && isfinite(E);
          q[DQ_NONFINITE] += fin ? 0.0 : 1.0;
        }
      }
      continue;
    }

    if constexpr (MODE == RM_XK) {
      // Kinematic run: the induction flux e = u x B and the status.
      // Inputs: 0 rho, 1-3 m, 4-6 B, 7 E.  Outputs: 0-2 e.
      const T gm1 = T(a.gamma[mem] - 1.0), gam = T(a.gamma[mem]);
      for (int x = tid; x < N; x += NT) {
        cx<T> v[8], o[3];
#pragma unroll
        for (int f = 0; f < 8; ++f) v[f] = buf[at(f, x)];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          auto g = [&](int f) -> T { return h == 0 ? v[f].x : v[f].y; };
          const T rho = g(0), mx = g(1), my = g(2), mz = g(3), Bx = g(4), By = g(5), Bz = g(6), E = g(7);
          const T ir = recip_(rho);
          const T ux = mx * ir, uy = my * ir, uz = mz * ir;
          const T B2 = Bx * Bx + By * By + Bz * Bz;
          const T P = gm1 * (E - T(0.5) * (mx * ux + my * uy + mz * uz) - T(0.5) * B2);
          const T e[3] = {uy * Bz - uz * By, uz * Bx - ux * Bz, ux * By - uy * Bx};
#pragma unroll
          for (int k = 0; k < 3; ++k) {
            if (h == 0) o[k].x = e[k];
            else o[k].y = e[k];
          }
          const T c = fmax(fabs(ux), fmax(fabs(uy), fabs(uz))) + sqrt_((gam * P + B2) * ir);
          if (!(c <= cfl)) cfl = c;  // NaN propagates
          const bool fin = finite_(rho) && finite_(mx) && finite_(my) && finite_(mz) && finite_(Bx) &&
                           finite_(By) && finite_(Bz) && finite_(E);
          bad += fin ? 0 : 1;
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) buf[at(k, x)] = o[k];
      }
    }

    if constexpr (MODE == RM_XA || FLUX || from_real(MODE)) {
      // only k <= K and N - k are read
      if constexpr (REAL_REGS) {
        lds_fft<T, PL, NB, NT, 1, BS, -1, RMAP, LAY, K, 1>(buf, stw, tid, nout);
      } else {
        if constexpr (SPEC_IN) __syncthreads();
        lds_fft<T, PL, NB, NT, 1, BS, -1, RMAP, LAY, K>(buf, stw, tid, nout);
      }
      // unpack: X0[k] = (Z[k] + conj Z[N-k]) / 2, X1[k] = -i (Z[k] - conj Z[N-k]) / 2, k = 0..K,
      // stored doubled (2 X0, 2 X1): the forward y pass that reads these rows
      // applies the 1/2 with its copy coefficient (an exact power-of-two
      // scaling, so the values are the same)
      T* out0 = member_ptr(a.out0, mem, a.bt.mstride);
      const int64_t ost = a.out_stride;
      auto unpack = [&](int fld, int k) {
        const cx<T> zk = buf[at(fld, k)];
        const cx<T> zm = buf[at(fld, k == 0 ? 0 : N - k)];
        const cx<T> x0 = mk<T>(zk.x + zm.x, zk.y - zm.y);
        const cx<T> x1 = mk<T>(zk.y + zm.y, zm.x - zk.x);
        T* dst = out0 + 2 * fld * ost;
        st(dst, row0 * PY + k, x0);
        st(dst, (row0 + 1) * PY + k, x1);
      };
      // the same with the field's output row as one wave-uniform pointer
      auto unpack_row = [&](cx<T>* dst, int fld, int k) {
        const cx<T> zk = buf[at(fld, k)];
        const cx<T> zm = buf[at(fld, k == 0 ? 0 : N - k)];
        dst[k] = mk<T>(zk.x + zm.x, zk.y - zm.y);
        dst[PY + k] = mk<T>(zk.y + zm.y, zm.x - zk.x);
      };
      if constexpr (WAVE) {
        // Each wave unpacks the fields it transformed, field by field: the
        // field and its output row are wave-uniform (scalar registers), so an
        // element costs its two LDS addresses and the store offset.  The flux
        // pass at N <= 256 (at most two 64-wide sweeps of a field) also
        // unrolls the sweeps, keeping the LDS addresses in registers across
        // row pairs; elsewhere that would cost occupancy.
        constexpr int W = NT / 64;
        constexpr int KIT = (NH + 63) / 64;
        const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
        cx<T>* const row_out = reinterpret_cast<cx<T>*>(out0) + row0 * PY;
#pragma unroll 1
        for (int fl = 0; fl < seqs_per_wave<NB, NT>(); ++fl) {
          const int fld = fl * W + wv;
          if (fld >= nout) break;
          cx<T>* const dst = row_out + fld * ost;
          if constexpr (is_flux(MODE) && KIT <= 2) {
#pragma unroll
            for (int it = 0; it < KIT; ++it) {
              const int k = (tid & 63) + 64 * it;
              if ((it + 1) * 64 <= NH || k < NH) unpack_row(dst, fld, k);
            }
          } else {
#pragma unroll 1
            for (int k = tid & 63; k < NH; k += 64) unpack_row(dst, fld, k);
          }
        }
      } else {
        for (int e = tid; e < nout * NH; e += NT) unpack(e / NH, e - (e / NH) * NH);
      }
    }
  }

  if constexpr (FLUX) {
    if (cur_m >= 0 && a.status) flush_status<NT>(double(cfl), bad, member_ptr(a.status, cur_m, a.bt.mstride), red);
  }
  if constexpr (MODE == RM_XDIAG) {
    for (int i = 0; i < kDiagQ; ++i) {
      const bool is_max = i == DQ_DIVB_MAX || i == DQ_CFL_MAX;
      const double r = is_max ? block_reduce<NT>(q[i], true, red, tid) : block_sum_comp<NT>(q[i], qc[i], red, tid);
      if (tid == 0) a.partials[(int64_t)blockIdx.x * kDiagQ + i] = r;
    }
  }
}

MHD_SCHED_END
}  // namespace mhd
