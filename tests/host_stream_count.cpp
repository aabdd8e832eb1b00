// Host test of stream_count.h: contexts of several devices, null streams among them.
#include "../paper_1412_4944_amd/csrc/stream_count.h"

#include <cstdio>

static int failures = 0;
static void expect(int got, int want, const char* what) {
    if (got != want) {
        std::printf("%s: %d, not %d\n", what, got, want);
        ++failures;
    }
}

int main() {
    sbo::StreamCount c;
    int a, b;
    expect(c.streams(0), 0, "nothing live");
    c.add(0, nullptr);
    c.add(0, nullptr);
    expect(c.streams(0), 1, "two contexts on one stream");
    c.add(1, nullptr);
    expect(c.streams(0), 1, "the null stream of another device does not count here");
    expect(c.streams(1), 1, "and counts there");
    c.add(1, &a);
    c.add(1, &b);
    expect(c.streams(0), 1, "streams of another device");
    expect(c.streams(1), 3, "three streams");
    c.remove(0, nullptr);
    expect(c.streams(0), 1, "one of two contexts gone");
    c.remove(0, nullptr);
    expect(c.streams(0), 0, "both gone");
    expect(c.streams(1), 3, "the other device is as it was");
    c.remove(1, &a);
    c.remove(1, &a);                           // not there: nothing happens
    expect(c.streams(1), 2, "one less");
    if (failures == 0) std::printf("ok\n");
    return failures != 0;
}
