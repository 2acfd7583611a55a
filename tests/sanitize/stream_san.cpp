// Driver that runs the read-backs' history (csrc/ifx_stream.hpp) under AddressSanitizer and UndefinedBehaviorSanitizer: which
// read-backs of a sequence of calls stream past the caches.  Compiled and run by tests/test_sanitizers.py.
#include <cstdint>
#include <cstdio>
#include <thread>
#include <vector>

#include "../../paper_2511_20714_amd/csrc/ifx_stream.hpp"

constexpr int64_t LINE = ifx::STREAM_FROM;
struct cache {
    int layers;
    int64_t bytes;  // that a read-back of a layer moves
    ifx::read_history h;
    cache(int l, int64_t b) : layers(l), bytes(b) { h.init(l); }
    bool read(int layer) { return h.read(layer, bytes, bytes * layers); }
};
static int bad = 0;
static void expect(const char *what, bool ok)
{
    if (!ok) std::printf("%s\n", what);
    bad |= !ok;
}

int main()
{
    const int64_t layer = 55 << 20;  // 4680 tokens of 12 heads, bf16
    {
        cache c(30, layer);
        bool all = true;
        for (int pass = 0; pass < 3; ++pass)
            for (int l = 0; l < 30; ++l)
                if (pass || l) all &= c.read(l);
                else expect("the first read-back of all", !c.read(l));
        expect("every layer in turn", all);
        bool any = c.read(0) && c.read(0);
        for (int i = 0; i < 20; ++i) any |= c.read(0);
        expect("one layer again and again", !any);
        any = false;
        for (int i = 0; i < 20; ++i) any |= c.read(1 + (i & 1)) && i >= 2;  // (the first two were read long ago)
        expect("two layers in turn", !any);
        c.h.attended(7, layer / 2);
        c.read(12);
        expect("attention has just read it", !c.read(7));
        for (int l = 0; l < 30; ++l) c.h.attended(l, layer / 2);
        c.read(29);
        expect("attention has read all since", c.read(0));
    }
    {
        cache c(30, layer);
        bool any = false;
        for (int pass = 0; pass < 2; ++pass)
            for (int l = 0; l < 30; ++l)
                for (int i = 0; i < 2; ++i) any |= c.read(l);
        expect("every layer twice", !any);
    }
    {
        cache c(5, layer);  // 275 MiB: the caches can hold all, or nearly
        bool any = false;
        for (int i = 0; i < 50; ++i) any |= c.read(i % 5);
        expect("layers that fit", !any);
        cache d(6, layer);
        for (int i = 0; i < 2; ++i) d.read(i);
        bool all = true;
        for (int i = 2; i < 50; ++i) all &= d.read(i % 6);
        expect("one layer more", all);
    }
    {
        cache at(1, LINE), past(1, LINE + 1), sum(3, LINE / 3);
        expect("a layer at the line", !at.read(0) && !at.read(0));
        expect("a layer past it", past.read(0) && past.read(0));
        bool any = false;
        for (int i = 0; i < 12; ++i) any |= sum.read(i % 3);
        expect("layers at the line", !any);
    }
    {
        cache c(30, layer);
        std::vector<std::thread> t;
        for (int k = 0; k < 4; ++k)
            t.emplace_back([&c, k] {
                for (int i = 0; i < 3000; ++i) (i + k) % 3 ? c.h.attended((i * 7 + k) % 30, c.bytes / 2) : (void)c.read((i + k) % 30);
            });
        for (auto &x : t) x.join();
        bool all = true;
        for (int i = 0; i < 60; ++i) all &= c.read(i % 30) || i < 30;
        expect("after calls at once", all);
    }
    std::printf(bad ? "FAILED\n" : "ok\n");
    return bad;
}
