// Host check of how the whole-column mixer deals out its work (compiled for the host only).  Groups of heads: none exceeds the
// scratch, there are as few as that allows, and, where the scratch holds whole eights, the eight XCDs get as even a share as
// without groups.  Lines: every one in exactly one workgroup, and the compute units of an XCD within one line of each other.
#include <cstdio>
#include <vector>

#include "mix_line.h"

using namespace spectre;

static bool groups_ok(int BH, int most) {
    const int c = line_group_heads(BH, most);
    int groups = 0, heads = 0;                                      // heads on the XCD that has most
    for (int bh0 = 0; c > 0 && bh0 < BH; bh0 += c) {
        groups += 1;
        heads += ((BH - bh0 < c ? BH - bh0 : c) + 7) / 8;
    }
    return c >= 1 && c <= most && groups == (BH + most - 1) / most && (most % 8 || heads == (BH + 7) / 8);
}

static bool lines_ok(int L, int nbh) {
    const int wgs = line_workgroups(L, nbh), units = 32;
    std::vector<int> seen((size_t)nbh * 32, 0);
    if (wgs < 1 || wgs > (L == 8192 ? 2 : 1) * units) return false;
    for (int xcd = 0; xcd < 8; ++xcd) {
        std::vector<int> load(units, 0);
        for (int j = 0; j < wgs; ++j) {
            const LineShare s = line_share(xcd, j, wgs, nbh);
            load[j % units] += s.count;
            for (int n = s.first; n < s.first + s.count; ++n) {
                const int head = 8 * (n / 32) + xcd;
                if (n < 0 || head >= nbh) return false;
                seen[(size_t)head * 32 + n % 32] += 1;
            }
        }
        int low = load[0], high = load[0];
        for (int x : load) {
            low = x < low ? x : low;
            high = x > high ? x : high;
        }
        if (high - low > 1) return false;
    }
    for (int x : seen)
        if (x != 1) return false;
    return true;
}

int main() {
    int failures = 0, cases = 0;
    for (int most = 1; most <= 260; ++most)
        for (int BH = 1; BH <= 1100; ++BH, ++cases)
            if (!groups_ok(BH, most) && failures++ < 10) std::printf("groups: most=%d BH=%d\n", most, BH);
    for (int L : {8192, 16384})
        for (int nbh = 1; nbh <= 400; ++nbh, ++cases)
            if (!lines_ok(L, nbh) && failures++ < 10) std::printf("lines: L=%d nbh=%d\n", L, nbh);
    std::printf("%d cases, %d failures\n", cases, failures);
    return failures ? 1 : 0;
}
