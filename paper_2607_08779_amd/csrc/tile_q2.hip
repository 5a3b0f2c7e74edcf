// Kernels of the matmul for middle token counts, 2-bit codes.
#include "tile_kernels.h"

namespace ssq {
namespace tile {

hipError_t launch_q2(const stream::StreamArgs& a, int kind, int form) { return tile_q<2>(a, kind, form); }

}  // namespace tile
}  // namespace ssq
