// Exact draws where there is little memory, and on a capturing stream: the sums of
// 16 amplitudes (1/16 of the state) are kept only where there is room for them.
// What the call accepts is what it accepts without them.
#include "fake_hip.h"

#include <cstdint>
#include <cstdio>

#include "../include/sv.h"

static int failures = 0;
static void check(bool ok, const char* what)
{
    if (ok) return;
    std::printf("%s\n", what);
    ++failures;
}

int main()
{
    const int n = 20;
    const int64_t shots = 5000;                     // more than a draw per 880 amplitudes: the sums pay
    const size_t state = (size_t)8 << n, sums = (size_t)8 << (n - 4), draws = (size_t)shots * 16, small = 100000;
    double u;
    int64_t out;
    const char *with = "k_shot_resolve_chunkedILb1E", *without = "k_shot_resolve_chunkedILb0E";
    auto draw = [&](sv_state s, int64_t count) {
        launched.clear();
        allocations = 0;
        return sv_sample_exact(s, 0, &u, count, &out);
    };
    sv_state s = nullptr;
    check(sv_alloc(n, 1, nullptr, nullptr, &s) == SV_OK, "sv_alloc");
    check(draw(s, shots) == SV_OK && was_launched(with) && !was_launched(without), "room enough: with the sums");
    check(sv_free(s) == SV_OK, "sv_free");
    // room for everything but the sums
    memory_limit = state + draws + small;
    check(memory_limit < state + draws + sums, "the limit lies below the sums");
    check(sv_alloc(n, 1, nullptr, nullptr, &s) == SV_OK, "sv_alloc");
    check(draw(s, shots) == SV_OK && was_launched(without) && !was_launched(with), "no room for the sums: without them");
    frees = 0;
    check(draw(s, shots) == SV_OK && was_launched(without) && frees == 0, "again: the scratch held stays");
    // held memory that is enough without them: captured, nothing is allocated
    capturing = true;
    check(draw(s, shots) == SV_OK && was_launched(without) && allocations == 0, "captured, without the sums");
    capturing = false;
    another_captures = true;
    check(draw(s, shots) == SV_OK && was_launched(without) && allocations == 0, "another stream captures, without the sums");
    another_captures = false;
    // room comes: with them, and then also captured
    memory_limit = ~size_t(0);
    check(draw(s, shots) == SV_OK && was_launched(with), "room again: with the sums");
    capturing = true;
    check(draw(s, shots) == SV_OK && was_launched(with) && allocations == 0, "captured, with the sums");
    capturing = false;
    check(sv_free(s) == SV_OK, "sv_free");
    // no room for the draws themselves: refused as ever
    memory_limit = state + small - 10000;            // the blocks and chunks take 71 KB
    check(sv_alloc(n, 1, nullptr, nullptr, &s) == SV_OK, "sv_alloc");
    check(draw(s, shots) == SV_ERR_OUT_OF_MEMORY && launched.empty(), "no room for the draws: out of memory");
    check(draw(s, 100) == SV_OK && was_launched(without), "few draws: without the sums");
    check(sv_free(s) == SV_OK && memory_held == 0, "sv_free");
    return failures ? 1 : 0;
}
