// How long a launch takes whose workgroups differ in length: a model for the dispatch rules (host only).
#ifndef LOZA_SSA_SCHEDULE_H
#define LOZA_SSA_SCHEDULE_H

#include <algorithm>

namespace loza {

// Workgroups go to the eight XCDs round-robin by number and there, in order, to the next of 32 compute units with
// room, which holds one or two; each of two runs at `shared` of its speed alone. `take` gives the time that one
// XCD's next workgroup takes alone, 0 after the last. Returns when its last one ends.
template <typename Take>
float xcd_time(int per_cu, float shared, Take &&take)
{
    // per compute unit: what its workgroups have left at time `at`, and when the first of them is done
    float left[2][32] = {}, at[32] = {}, next[32];
    auto speed = [&](int c) { return left[0][c] > 0.f && left[1][c] > 0.f ? shared : 1.f; };
    auto due = [&](int c) {
        const float a = left[0][c], b = left[1][c], first = a > 0.f && (b <= 0.f || a < b) ? a : b;
        next[c] = first > 0.f ? at[c] + first / speed(c) : 0.f;
    };
    for (int slot = 0; slot < per_cu; ++slot)
        for (int c = 0; c < 32; ++c) left[slot][c] = take();
    for (int c = 0; c < 32; ++c) due(c);
    for (float w = take(); w > 0.f; w = take()) {
        const int c = (int)(std::min_element(next, next + 32) - next);
        int s = left[0][c] <= 0.f ? 0 : per_cu == 2 && left[1][c] <= 0.f ? 1 : -1;   // a place that is free already
        if (s < 0) {
            const float done = (next[c] - at[c]) * speed(c);
            at[c] = next[c];
            s = left[1][c] > 0.f && left[1][c] < left[0][c] ? 1 : 0;
            left[s][c] = 0.f;
            left[1 - s][c] = left[1 - s][c] > done * 1.0001f ? left[1 - s][c] - done : 0.f;
        }
        left[s][c] = w;
        if (per_cu == 2 && left[1 - s][c] <= 0.f) next[c] = at[c] * 1.0001f;   // (both ended together; others first)
        else due(c);
    }
    float longest = 0.f;
    for (int c = 0; c < 32; ++c) {
        const float a = left[0][c], b = left[1][c], m = a < b ? a : b;   // two together, then the longer one alone
        const float end = at[c] + (m > 0.f ? m / shared : 0.f) + (a + b - 2.f * m);
        if (end > longest) longest = end;
    }
    return longest;
}

}  // namespace loza
#endif
