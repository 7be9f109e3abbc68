// Host check (built by tests/test_brick_rest_cpu.py): when a context launches
// bricks again after launches that ran on one workgroup.
#include <cstdio>
#include <vector>

#include "bricks.h"
using namespace ibmg;

// the solves of n that launch bricks; alone(k): such a launch of solve k runs on one workgroup
template <typename F>
static std::vector<int> tries(int n, F alone)
{
    BrickRest r;
    std::vector<int> out;
    int solo = 0;
    for (int k = 0; k < n; ++k) {
        r.solve_begins();
        bool tried = false;
        for (int it = 0; it < 3; ++it) {   // iterations
            if (!r.resting()) {
                tried = true;
                if (alone(k)) ++solo;
            }
            r.saw(solo);
        }
        if (tried) out.push_back(k);
    }
    return out;
}

int main()
{
    long long bad = 0;
    auto expect = [&](const char *what, const std::vector<int> &got, const std::vector<int> &want) {
        if (got == want) return;
        ++bad;
        printf("%s:", what);
        for (int k : got) printf(" %d", k);
        printf("\n");
    };
    std::vector<int> all(40);
    for (int k = 0; k < 40; ++k) all[k] = k;
    expect("never alone", tries(40, [](int) { return false; }), all);
    // one slow start: the next solve rests, then all is as before
    std::vector<int> once;
    for (int k = 0; k < 40; ++k)
        if (k != 6) once.push_back(k);
    expect("once", tries(40, [](int k) { return k == 5; }), once);
    // another process on the device for good: rests of 1, 2, 4, ... solves, 256 at most
    std::vector<int> always;
    for (int k = 0, rest = 1; k < 2000; k += rest + 1, rest = rest < 256 ? 2 * rest : 256) always.push_back(k);
    expect("always", tries(2000, [](int) { return true; }), always);
    // rests of 1 after 0, 2 after 2, 4 after 5; the next would be 8, halved as each of 11 to 13 begins after a good
    // solve, so 13 is followed by a rest of 1 and 11, had it been the bad one, by one of 4
    expect("seldom", tries(18, [](int k) { return k <= 5 || k == 13; }), {0, 2, 5, 10, 11, 12, 13, 15, 16, 17});
    expect("sooner", tries(18, [](int k) { return k <= 5 || k == 11; }), {0, 2, 5, 10, 11, 16, 17});
    printf("%lld mismatches\n", bad);
    return bad != 0;
}
