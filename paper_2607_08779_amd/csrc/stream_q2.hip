// Instantiations of the rounded streaming kernels for 2-bit codes.
#include "stream_kernels.h"

namespace ssq {
namespace stream {

hipError_t launch_rounded_q2(const StreamArgs& a, int kind, int tok, int rt) { return rounded_q<2>(a, kind, tok, rt); }

}  // namespace stream
}  // namespace ssq
