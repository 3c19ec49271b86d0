// Instantiates every pass kernel for one grid size N = MHD_N, both precisions
// (FP64 only up to N = 512, where the row pass's LDS footprint still fits).
#include "mhd_kernels.h"
#include "mhd_registry.h"
#include "mhd_slab.h"

#ifndef MHD_N
#error "compile with -DMHD_N=<grid size>"
#endif

namespace mhd {
namespace {

// Column passes: one instantiation per direction, term count, axis (z or y) and, where
// a launch chooses, way of storing.
template <typename T, int N, int S, int MAXT, bool MX, bool Z>
void col_axis(const ColArgs<T>& a, dim3 g, hipStream_t s) {
  constexpr ColStream cs = col_stream<N, S, MAXT, MX, Z>();
  const dim3 nt(col_threads<T, N, MX, S, MAXT, Z>());
  if constexpr (cs != CS_NEVER) {
    if (cs == CS_ALWAYS || a.stream) {
      hipLaunchKernelGGL((k_col<T, N, S, MAXT, MX, Z, true>), g, nt, 0, s, a);
      return;
    }
  }
  if constexpr (cs != CS_ALWAYS) hipLaunchKernelGGL((k_col<T, N, S, MAXT, MX, Z, false>), g, nt, 0, s, a);
}
template <typename T, int N, int S, int MAXT, bool MX>
void col_launch(const ColArgs<T>& a, dim3 g, hipStream_t s) {
  if (a.kind == PK_ZINV || a.kind == PK_ZFWD) col_axis<T, N, S, MAXT, MX, true>(a, g, s);
  else col_axis<T, N, S, MAXT, MX, false>(a, g, s);
}
template <typename T, int N, bool MX>
void col_inv(int maxt, const ColArgs<T>& a, dim3 g, hipStream_t s) {
  if (maxt <= 1) col_launch<T, N, 1, 1, MX>(a, g, s);
  else col_launch<T, N, 1, kMaxTerms, MX>(a, g, s);
}
template <typename T, int N, bool MX>
void col_fwd(const ColArgs<T>& a, dim3 g, hipStream_t s) {
  col_launch<T, N, -1, 1, MX>(a, g, s);
}
// Tile width and resident workgroups per CU of a column-pass class (both ways of
// storing come out at the same registers or within a few).
template <typename T, int N, int S, int MAXT, bool MX, bool Z>
ColClass col_occ(void) {
  ColClass c;
  c.width = col_tile<T, N, MX, S, MAXT, Z>();
  constexpr bool st = col_stream<N, S, MAXT, MX, Z>() == CS_ALWAYS;
  const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&c.blocks, k_col<T, N, S, MAXT, MX, Z, st>,
                                                                    col_threads<T, N, MX, S, MAXT, Z>(), 0);
  if (e != hipSuccess || c.blocks < 1) c.blocks = 1;
  // the 1024-thread tiles at 256: one workgroup per CU also where the registers
  // would let two reside (more rows of more fields in flight at once cost HBM
  // efficiency: 12-field forward y pass 239 us with one, 253 with two)
  if (N == 256 && col_threads<T, N, MX, S, MAXT, Z>() == 4 * kThreads) c.blocks = 1;
  return c;
}
template <typename T, int N, bool MX>
ColClass col_class(int dir, int maxt, bool z) {
  if (dir < 0) return z ? col_occ<T, N, -1, 1, MX, true>() : col_occ<T, N, -1, 1, MX, false>();
  if (maxt <= 1) return z ? col_occ<T, N, 1, 1, MX, true>() : col_occ<T, N, 1, 1, MX, false>();
  return z ? col_occ<T, N, 1, kMaxTerms, MX, true>() : col_occ<T, N, 1, kMaxTerms, MX, false>();
}
template <typename T, int N>
void rhs(const RhsArgs<T>& a, dim3 g, hipStream_t s) {
  hipLaunchKernelGGL((k_zfwd_rhs<T, N>), g, dim3(rhs_threads<T, N>()), 0, s, a);
}
template <typename T, int N>
void zyinv(const ColArgs<T>& a, int nmem, hipStream_t s) {
  hipLaunchKernelGGL((k_zyinv<T, N>), dim3((unsigned)(nmem * a.nout * Band<N>::NH)),
                     dim3(slab_threads<T, N>()), 0, s, a);
}
template <typename T, int N>
void yzfwd(const ColArgs<T>& a, int nmem, hipStream_t s) {
  hipLaunchKernelGGL((k_yzfwd<T, N>), dim3((unsigned)(nmem * a.nout * Band<N>::NH)),
                     dim3(slab_threads<T, N>()), 0, s, a);
}
template <typename T, int N>
void strain_rho(const ColArgs<T>& a, const UpdateArgs<T>& q, int nmem, hipStream_t s) {
  hipLaunchKernelGGL((k_strain_rho<T, N>), dim3((unsigned)(nmem * (a.nout + 1) * Band<N>::NH)),
                     dim3(kTeams * slab_threads<T, N>()), 0, s, a, q);
}
template <typename T, int N>
void yzrhs(const RhsArgs<T>& a, int nfrozen, int nmem, hipStream_t s) {
  hipLaunchKernelGGL((k_yzrhs<T, N>), dim3((unsigned)(nmem * (a.nf + nfrozen) * Band<N>::NH)),
                     dim3(kTeams * slab_threads<T, N>()), 0, s, a, nfrozen);
}
// fn<MODE>() for a run-time row mode
template <typename F>
void with_row_mode(int mode, F&& fn) {
  switch (mode) {
    case RM_XA: fn(std::integral_constant<int, RM_XA>()); break;
    case RM_XB: fn(std::integral_constant<int, RM_XB>()); break;
    case RM_XFWD_REAL: fn(std::integral_constant<int, RM_XFWD_REAL>()); break;
    case RM_XINV_REAL: fn(std::integral_constant<int, RM_XINV_REAL>()); break;
    case RM_XDIAG: fn(std::integral_constant<int, RM_XDIAG>()); break;
    case RM_XL: fn(std::integral_constant<int, RM_XL>()); break;
    case RM_XK: fn(std::integral_constant<int, RM_XK>()); break;
    case RM_XFWD_ONE: fn(std::integral_constant<int, RM_XFWD_ONE>()); break;
    case RM_XINV_ONE: fn(std::integral_constant<int, RM_XINV_ONE>()); break;
    default: break;
  }
}
template <typename T, int N>
void row(int mode, const RowArgs<T>& a, dim3 g, hipStream_t s) {
  with_row_mode(mode, [&](auto m) {
    constexpr int M = decltype(m)::value;
    hipLaunchKernelGGL((k_row<T, N, M>), g, dim3(row_threads<T, N, M>()), 0, s, a);
  });
}
template <typename T, int N>
int row_occupancy(int mode) {
  if (mode == RM_XFWD_ONE || mode == RM_XINV_ONE) {
    // one wave of at most 128 registers and its LDS; the runtime takes 50 us per kernel to
    // say the same when the first context of a size is made
    constexpr int lds = 2 * (int)sizeof(T) * (2 * N + N / 8 + 1);
    return 160 * 1024 / lds < 16 ? 160 * 1024 / lds : 16;
  }
  int blocks = 0;
  hipError_t e = hipSuccess;
  with_row_mode(mode, [&](auto m) {
    constexpr int M = decltype(m)::value;
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, k_row<T, N, M>, row_threads<T, N, M>(), 0);
  });
  return (e == hipSuccess && blocks > 0) ? blocks : 1;
}

// MX: the mixed path.  Its column passes run the radix-16 plans; the row passes,
// the z-RHS pass and the small grids run the FP32 kernels, which measured faster
// there (256: flux pass 512 -> 361 us, z-RHS 318 -> 235; 512: 4496 -> 2695 and
// 2329 -> 2031) and are more accurate.
template <typename T, int N, bool MX>
Kern<T> make() {
  Kern<T> k;
  k.n = N;
  k.rhs_width = rhs_tile<T, N>();
  k.twiddles = make_twiddles<T, PlanOf<N, MX>>;
  k.twiddles_valu = make_twiddles<T, PlanOf<N>>;
  k.col_inv = col_inv<T, N, MX>;
  k.col_fwd = col_fwd<T, N, MX>;
  k.rhs = rhs<T, N>;
  if constexpr (N <= kSlabMax && MHD_SCHED == 0) {
    k.zyinv = zyinv<T, N>;
    k.yzfwd = yzfwd<T, N>;
    k.strain_rho = strain_rho<T, N>;
    k.yzrhs = yzrhs<T, N>;
  }
  k.row = row<T, N>;
  k.row_occupancy = row_occupancy<T, N>;
  k.col_class = col_class<T, N, MX>;
  return k;
}

}  // namespace

#define MHD_CAT2(a, b) a##b
#define MHD_CAT(a, b) MHD_CAT2(a, b)
#if MHD_SCHED == 1
// the alternative schedule: FP32 only
void MHD_CAT(register_s1_, MHD_N)(Registry& r) { r.f32s1[MHD_N] = make<float, MHD_N, false>(); }
#else
void MHD_CAT(register_, MHD_N)(Registry& r) {
  r.f32[MHD_N] = make<float, MHD_N, false>();
  r.mx[MHD_N] = make<float, MHD_N, (MHD_N > kSlabMax)>();
#if MHD_N <= 512
  r.f64[MHD_N] = make<double, MHD_N, false>();
#endif
}
#endif

}  // namespace mhd
