// Instantiations of the exact streaming kernels (2- and 4-bit codes, up to 16 tokens).
#include "stream_kernels.h"

namespace ssq {
namespace stream {

hipError_t launch_exact(const StreamArgs& a, int q, int kind, int tok, int rt) {
  switch (q * 4 + kind) {
    case 8: return exact_any<2, kMetaNone>(a, tok, rt);
    case 9: return exact_any<2, kMetaZp>(a, tok, rt);
    case 10: return exact_any<2, kMetaMin>(a, tok, rt);
    case 16: return exact_any<4, kMetaNone>(a, tok, rt);
    case 17: return exact_any<4, kMetaZp>(a, tok, rt);
    case 18: return exact_any<4, kMetaMin>(a, tok, rt);
  }
  return hipErrorInvalidValue;
}

}  // namespace stream
}  // namespace ssq
