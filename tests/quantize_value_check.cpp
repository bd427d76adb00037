// csrc/quantize_value.h on the host, called from test_quantization_any_bits.py.
#include <hip/hip_runtime.h>

#include "quantize_value.h"

extern "C" void quantize(const float *x, const float *s, const float *mn, int n, int qmax, unsigned char *codes) {
    for (int i = 0; i < n; ++i) {
        const float r = s[i] != 0.0f ? 1.0f / s[i] : 0.0f;   // as token_scale_min
        codes[i] = (unsigned char)packkv::quantize_value(x[i], s[i], mn[i], r, qmax);
    }
}
