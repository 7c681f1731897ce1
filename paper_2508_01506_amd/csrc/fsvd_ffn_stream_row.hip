// The FFN core with wavefront-private weight streams for row-major weights: a translation unit of its own, so that these
// instantiations compile beside those for prepacked weights.
#define FSVD_FFN_STREAM_ROW 1
#include "fsvd_ffn_stream.hip"
