// Launchers of the line kernels for levels with few columns (line_block.h).

#include "line_block.h"

namespace gmg {

namespace {

template <typename T, int MODE, int CB>
hipError_t block_dispatch_cb(const Lvl<T>& L, const BlockArgs<T>& a, hipStream_t s) {
  const int ncols = L.nx * L.ny;
  const dim3 grid((unsigned)block_count(L.nx, L.ny)), block(kBlockThreads);
  const int half = (L.nz + 1) / 2;
  if (half <= 4)
    hipLaunchKernelGGL((k_line_block<T, MODE, 4, CB>), grid, block, 0, s, L, a, ncols);
  else if (half <= 8)
    hipLaunchKernelGGL((k_line_block<T, MODE, 8, CB>), grid, block, 0, s, L, a, ncols);
  else if (half <= 16)
    hipLaunchKernelGGL((k_line_block<T, MODE, 16, CB>), grid, block, 0, s, L, a, ncols);
  else if (half <= 32)
    hipLaunchKernelGGL((k_line_block<T, MODE, 32, CB>), grid, block, 0, s, L, a, ncols);
  else if (half <= 64)
    hipLaunchKernelGGL((k_line_block<T, MODE, 64, CB>), grid, block, 0, s, L, a, ncols);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

template <typename T, int MODE>
hipError_t block_dispatch(const Lvl<T>& L, const BlockArgs<T>& a, hipStream_t s) {
  switch (block_cols((int64_t)L.nx * L.ny)) {
    case 8:
      return block_dispatch_cb<T, MODE, 8>(L, a, s);
    case 16:
      return block_dispatch_cb<T, MODE, 16>(L, a, s);
    default:
      return block_dispatch_cb<T, MODE, 32>(L, a, s);
  }
}

}  // namespace

int block_cols(int64_t ncols) { return ncols <= 8 * 256 ? 8 : ncols <= 16 * 256 ? 16 : 32; }

int64_t block_count(int nx, int ny) {
  const int64_t ncols = (int64_t)nx * ny;
  const int cb = block_cols(ncols);
  return (ncols + cb - 1) / cb;
}

hipError_t launch_grouped_block(GKind kind, int half, int cb, const GItem<float>* items,
                                int nitems, int nblocks, const int* active, float rho,
                                hipStream_t s) {
  const dim3 grid(nblocks), block(kBlockThreads);
#define GMG_GBLOCK(OP, H, CB)                                                                  \
  if (half == H && cb == CB) {                                                                 \
    hipLaunchKernelGGL((k_line_block_grouped<(int)BlockOp::OP, H, CB>), grid, block, 0, s,     \
                       items, nitems, active, rho);                                            \
    return hipGetLastError();                                                                  \
  }
#define GMG_GBLOCKS(OP)                                                                 \
  GMG_GBLOCK(OP, 4, 8) GMG_GBLOCK(OP, 8, 8) GMG_GBLOCK(OP, 16, 8) GMG_GBLOCK(OP, 32, 8) \
  GMG_GBLOCK(OP, 64, 8) GMG_GBLOCK(OP, 4, 16) GMG_GBLOCK(OP, 8, 16)                     \
  GMG_GBLOCK(OP, 16, 16) GMG_GBLOCK(OP, 32, 16) GMG_GBLOCK(OP, 64, 16)                  \
  GMG_GBLOCK(OP, 4, 32) GMG_GBLOCK(OP, 8, 32) GMG_GBLOCK(OP, 16, 32)                    \
  GMG_GBLOCK(OP, 32, 32) GMG_GBLOCK(OP, 64, 32)
  switch (kind) {
    case GKind::SMOOTH:
      GMG_GBLOCKS(SMOOTH)
      break;
    case GKind::PROLONG_SMOOTH:
      GMG_GBLOCKS(PROLONG_SMOOTH)
      break;
    case GKind::RESTRICT_SOLVE:
      GMG_GBLOCKS(RESTRICT_SOLVE)
      break;
    default:
      break;
  }
#undef GMG_GBLOCKS
#undef GMG_GBLOCK
  return hipErrorInvalidValue;
}

template <typename T>
hipError_t launch_block(BlockOp op, const Lvl<T>& L, const BlockArgs<T>& a, hipStream_t s) {
  switch (op) {
    case BlockOp::SOLVE:
      return block_dispatch<T, (int)BlockOp::SOLVE>(L, a, s);
    case BlockOp::SMOOTH:
      return block_dispatch<T, (int)BlockOp::SMOOTH>(L, a, s);
    case BlockOp::SMOOTH_NORM:
      return block_dispatch<T, (int)BlockOp::SMOOTH_NORM>(L, a, s);
    case BlockOp::PROLONG_SMOOTH:
      return block_dispatch<T, (int)BlockOp::PROLONG_SMOOTH>(L, a, s);
    case BlockOp::RESTRICT_SOLVE:
      return block_dispatch<T, (int)BlockOp::RESTRICT_SOLVE>(L, a, s);
    case BlockOp::CG:
      if constexpr (sizeof(T) == 8) return block_dispatch<T, (int)BlockOp::CG>(L, a, s);
  }
  return hipErrorInvalidValue;
}

template hipError_t launch_block<double>(BlockOp, const Lvl<double>&, const BlockArgs<double>&,
                                         hipStream_t);
template hipError_t launch_block<float>(BlockOp, const Lvl<float>&, const BlockArgs<float>&,
                                        hipStream_t);

}  // namespace gmg
