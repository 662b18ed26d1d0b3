// Host build of arithmetic that the kernels take from their headers, for CPU
// tests: each function applies the header's own code to arrays of inputs.
#include "../../paper_1312_3004_amd/csrc/rewl_replay.h"

extern "C" {

// n[i] additions of l[i] to x[i]; returns how many took the closed form.
size_t replay_binary64_all(size_t count, double *x, const double *l, const uint32_t *n)
{
    size_t closed = 0;
    for (size_t i = 0; i < count; ++i) {
        if (rewl_gpu::replay_binary64(x[i], l[i], n[i])) {
            ++closed;
            continue;
        }
        for (uint32_t k = 0; k < n[i]; ++k) x[i] = x[i] + l[i];
    }
    return closed;
}

// The same for pairs; returns how many additions were made one by one.
size_t replay_pair_all(size_t count, float *hi, float *lo, const float *l, const uint32_t *n)
{
    size_t single = 0;
    for (size_t i = 0; i < count; ++i)
        rewl_gpu::replay_pair(hi[i], lo[i], l[i], n[i], [&](bool more) {
            single += more;
            return more;
        });
    return single;
}

}
