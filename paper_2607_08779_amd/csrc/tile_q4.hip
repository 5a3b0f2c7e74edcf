// Kernels of the matmul for middle token counts, 4-bit codes.
#include "tile_kernels.h"

namespace ssq {
namespace tile {

hipError_t launch_q4(const stream::StreamArgs& a, int kind, int form) { return tile_q<4>(a, kind, form); }

}  // namespace tile
}  // namespace ssq
