// Instantiations of the rounded streaming kernels for 4-bit codes.
#include "stream_kernels.h"

namespace ssq {
namespace stream {

hipError_t launch_rounded_q4(const StreamArgs& a, int kind, int tok, int rt) { return rounded_q<4>(a, kind, tok, rt); }

}  // namespace stream
}  // namespace ssq
