// Host build of arithmetic that the kernels take from their headers, for CPU
// tests: each function applies the header's own code to arrays of inputs.
#include "../../paper_1312_3004_amd/csrc/rewl_handover.h"
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

// Records written and read by the two sides of a hand-over of n attempts: rows
// of (barriers passed, record, block), at most `max` of each; the counts and
// the barriers of either side go to out[0 .. 3].
void handover_trace(int64_t n, size_t max, int64_t *written, int64_t *read, int64_t *out)
{
    int64_t wrote = 0, got = 0, wsync = 0, rsync = 0;
    auto put = [&](int64_t *to, int64_t &at, int64_t when, int64_t base) {
        if ((size_t)at >= max) return;
        to[3 * at] = when;
        to[3 * at + 1] = rewl_gpu::handover_slot(base);
        to[3 * at++ + 2] = base / 64;
    };
    rewl_gpu::handover_draw(n, [&](int64_t base) { put(written, wrote, wsync, base); }, [&] { ++wsync; });
    auto fetch = [&](int64_t base) { put(read, got, rsync, base); };
    rewl_gpu::handover_decide(n, fetch, [&] { ++rsync; }, [&](int64_t base) { fetch(base + 64); });
    out[0] = wrote;
    out[1] = got;
    out[2] = wsync;
    out[3] = rsync;
}

}
