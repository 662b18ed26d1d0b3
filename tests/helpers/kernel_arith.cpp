// Host build of arithmetic that the kernels take from their headers, for CPU
// tests: each function applies the header's own code to arrays of inputs.
#include "../../paper_1312_3004_amd/csrc/rewl_handover.h"
#include "../../paper_1312_3004_amd/csrc/rewl_moves.h"
#include "../../paper_1312_3004_amd/csrc/rewl_replay.h"
#include "../../paper_1312_3004_amd/csrc/rewl_slots.h"

#include <atomic>
#include <cstdlib>
#include <thread>
#include <vector>

namespace {

// Squared distance on the 16-bit grid, as the kernels' dot products of 16-bit
// differences give it.
uint32_t grid2(rewl_gpu::MoveGrid a, rewl_gpu::MoveGrid b)
{
    auto d = [](uint32_t x, uint32_t y) { return (int32_t)(int16_t)(uint16_t)(x - y); };
    auto sq = [](int32_t v) { return (uint32_t)(v * v); };
    return sq(d(a.xy & 0xffffu, b.xy & 0xffffu)) + sq(d(a.xy >> 16, b.xy >> 16)) + sq(d(a.z, b.z));
}

}  // namespace

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

// The partner screens.  Bead i moves from o[i] by the displacement of the words
// r[i] and the partner is at q[i] (3 numbers a place, in [0, box)).  Bits of
// kept[i]: 0 / 1 the partner is within the cut-off of the old / new place,
// 2 the screen of a displacement keeps it, 3 that of a reptation (old place)
// keeps it, 4 the correction test of two displacements (the partner moves too,
// by the words r2[i]) holds, 5 the moved partner is within the cut-off of
// either place of the bead.
void screen_all(size_t count, const float *o, const uint32_t *r, const float *q, const uint32_t *r2, float box,
                uint8_t *kept)
{
    using namespace rewl_gpu;
    const float scale = 65536.0f / box, half = 0.5f * box;
    for (size_t i = 0; i < count; ++i) {
        const float *a = o + 3 * i, *b = q + 3 * i;
        float d[3], e[3], n[3], m[3];
        for (int c = 0; c < 3; ++c) {
            d[c] = move_disp(r[3 * i + c]);
            e[c] = move_disp(r2[3 * i + c]);
            n[c] = move_wrap(a[c] + d[c], box);
            m[c] = move_wrap(b[c] + e[c], box);
        }
        const float reach = move_reach(d[0], d[1], d[2], box), reach2 = move_reach(e[0], e[1], e[2], box);
        const uint32_t g = grid2(move_grid(b, scale), move_grid(a, scale));
        const double cut2 = 6.25;
        kept[i] = (uint8_t)((move_r2(a, b, box, half) < cut2) | (move_r2(n, b, box, half) < cut2) << 1 |
                            (g <= move_grid_limit(2.5f + reach, scale)) << 2 |
                            (g <= move_grid_limit(2.5f + move_slack(box), scale)) << 3 |
                            (g <= move_grid_limit(2.5f + reach + reach2, scale)) << 4 |
                            (move_r2(a, m, box, half) < cut2 || move_r2(n, m, box, half) < cut2) << 5);
    }
}

// Entry r of the corrections that `lane` of a workgroup of `waves` wavefronts
// reads, from a table whose entry i is i + 1; *last: the furthest entry read.
int64_t correction_read(int lane, int waves, int r, int64_t *last)
{
    struct Table {
        int64_t *last;
        int64_t operator[](int i) const
        {
            if (i > *last) *last = i;
            return i + 1;
        }
    };
    *last = -1;
    return rewl_gpu::move_corrections(Table{last}, lane, waves)[r];
}

// Workgroup of the continuous models: wavefronts, 16-bit places kept, LDS bytes.
void move_workgroup(size_t used, size_t per_wave, int particles, int walkers, int64_t *out)
{
    const rewl_gpu::MovePlan p = rewl_gpu::move_plan(used, per_wave, particles, walkers);
    out[0] = p.waves;
    out[1] = p.grid;
    out[2] = (int64_t)p.lds;
}

// The shared slots: 0 if a block that could not be allocated gives none, the
// block is allocated once, its slots are distinct and all used before none is
// left, and a slot given back is taken again; else the number of the failed step.
int slots_in_order(void)
{
    rewl_host::SlotBlock block;
    int calls = 0;
    unsigned char *mem = nullptr;
    block.reserve([&](size_t) -> void * { ++calls; return nullptr; });
    if (block.take()) return 1;
    for (int i = 0; i < 3; ++i)
        block.reserve([&](size_t bytes) -> void * { ++calls; return mem = (unsigned char *)malloc(bytes); });
    if (calls != 2) return 2;
    std::vector<unsigned char *> slot;
    while (unsigned char *s = block.take()) slot.push_back(s);
    if (slot.size() != 64) return 3;
    for (size_t i = 0; i < slot.size(); ++i)
        if (slot[i] != mem + i * rewl_host::SlotBlock::kBytes) return 4;
    block.give(nullptr);
    block.give(slot[17]);
    block.give(slot[40]);
    if (block.take() != slot[17] || block.take() != slot[40] || block.take()) return 5;
    free(mem);
    return 0;
}

// Threads that take and give slots: how often one was found taken twice.
int slots_shared(int threads, int rounds)
{
    rewl_host::SlotBlock block;
    std::vector<unsigned char> mem(64 * rewl_host::SlotBlock::kBytes);
    std::atomic<int> owner[64] = {}, clashes{0};
    std::vector<std::thread> pool;
    for (int t = 0; t < threads; ++t)
        pool.emplace_back([&] {
            for (int i = 0; i < rounds; ++i) {
                block.reserve([&](size_t) -> void * { return mem.data(); });
                unsigned char *held[12];
                for (auto &s : held) {
                    s = block.take();
                    if (s && owner[(s - mem.data()) / rewl_host::SlotBlock::kBytes].exchange(1)) ++clashes;
                }
                for (auto &s : held) {
                    if (s) owner[(s - mem.data()) / rewl_host::SlotBlock::kBytes] = 0;
                    block.give(s);
                }
            }
        });
    for (auto &t : pool) t.join();
    return clashes;
}

double pair_decision_margin(double M, double d, float lo) { return rewl_gpu::pair_margin(M, d, lo); }

int correction_entries(int waves) { return rewl_gpu::move_table(waves); }

}
