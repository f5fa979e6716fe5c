// Constant-Q kernels tap by tap: the launches of nna_short.h.
#include "nna_short.h"

namespace nna {
namespace {

template <int FB, int WK, int LAYOUT>
__global__ __launch_bounds__(256, LAYOUT != COLUMNS ? 3 : WK == 1 ? 4 : 2) void short_kernel(const ShortParams P) {
  extern __shared__ __attribute__((aligned(16))) unsigned short S[];
  // the items of one tile are neighbours on one XCD
  const int n_items = P.n_items;
  const long long local = blockIdx.x >> 3, per_xcd = (P.n_ft + 7) >> 3, tile = local / n_items;
  const long long ft = (blockIdx.x & 7) * per_xcd + tile;
  if (tile >= per_xcd || ft >= P.n_ft) return;
  const ShortItem item = P.items[local - tile * n_items];
  short_tile<FB, WK, LAYOUT, SHORT_SCALE>(P, item, ft, S);
}

template <int FB, int WK, int LAYOUT>
struct Form {
  static hipError_t allow_lds() {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(short_kernel<FB, WK, LAYOUT>), hipFuncAttributeMaxDynamicSharedMemorySize, SHORT_LDS);
  }
  static void launch(const ShortParams& p, unsigned blocks, hipStream_t stream) {
    hipLaunchKernelGGL((short_kernel<FB, WK, LAYOUT>), dim3(blocks), dim3(256), (size_t)p.plane * 6 + 16, stream, p);
  }
};

// calls fn with the kernel of a form of nna_internal.h
template <typename Fn>
void with_form(int form, bool octets, Fn fn) {
  if (form == SHORT_64) octets ? fn(Form<4, 4, OCTETS_OF>{}) : fn(Form<4, 4, QUADS_OF>{});
  else if (form == SHORT_32) octets ? fn(Form<2, 4, OCTETS_OF>{}) : fn(Form<2, 4, QUADS_OF>{});
  else if (form == SHORT_16) octets ? fn(Form<1, 4, OCTETS_OF>{}) : fn(Form<1, 4, QUADS_OF>{});
  else if (form == SHORT_COLUMNS) fn(Form<2, 1, COLUMNS>{});
  else fn(Form<4, 4, COLUMNS>{});
}

}  // namespace

hipError_t short_kernels_init() {
  hipError_t e = hipSuccess;
  for (int form = 0; form < SHORT_FORMS; ++form)
    for (const bool octets : {true, false})
      with_form(form, octets, [&](auto f) { if (e == hipSuccess) e = f.allow_lds(); });
  return e;
}

hipError_t launch_cqt_short(const ShortParams& p, hipStream_t stream) {
  clear_stale_error();
  const long long blocks = (p.n_ft + 7) / 8 * 8 * p.n_items;
  if (blocks <= 0 || blocks > 0x7fffffffLL || p.g.L < 4 || p.g.hop % 4 != 0) return hipErrorInvalidValue;
  if (p.form < 0 || p.form >= SHORT_FORMS || p.tile_frames < 1 || p.tile_frames > SHORT_FRAMES[p.form]) return hipErrorInvalidValue;
  if (p.form == SHORT_COLUMNS_64 && p.columns_at_once != 32 && p.columns_at_once != 64 && p.columns_at_once != 128) return hipErrorInvalidValue;
  if (p.plane % 8 != 0 || p.plane < SHORT_PLANE_MIN[p.form] || (size_t)p.plane * 6 + 16 > (size_t)SHORT_LDS) return hipErrorInvalidValue;
  with_form(p.form, p.octets != 0, [&](auto f) { f.launch(p, (unsigned)blocks, stream); });
  return hipGetLastError();
}

}  // namespace nna
