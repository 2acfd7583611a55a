// What streams past the caches (non-temporal accesses), decided on the host.  Pure host integer code, no device calls.
//
// Plain stores leave a commit's destination in the caches, where the attention call after it finds it, and its source
// stays there for whoever reads it again.  Only of what the memory-side cache cannot hold is nothing found later, and there
// the dirty lines are in the way: a commit launch that moves more than it holds (commit_streams) streams on both sides.
// us, plain -> streaming, above the line: 30 layers of 4680 tokens x 12 heads 315 -> 297, fp32 20 layers of 2000 x 8 committed and
// read back 301 -> 276, attention and commit of 10 layers of 3600 x 12 1631 -> 1615, of 6 of 1560 x 40 and of 30 of 1560 x
// 12 level; below it, attention and commit: 4 layers of 480 x 12 77.6 -> 85.0, 2 of 776 x 8 38.5 -> 40.5, 2 of 1560 x 24 195 -> 204,
// 12 of 720 x 20 498 -> 509.  The line lies a little above the cache's 256 MiB: 5 layers of 4680 x 12 (274 MiB) committed and
// read back 111 -> 113, 6 (329) 148 -> 135, fp32 10 of 2000 x 8 (313) 143 -> 137.
//
// A read-back's source streams (read_history) where it cannot be in the caches and nobody is likely to want it there.  us a layer
// of 30 of 4680 x 12, plain -> streaming, bf16 and fp8 cache: every layer read in turn 14.0 -> 12.7, 11.4 -> 10.5, each
// committed just before 25.5 -> 23.4, 20.7 -> 20.2, all committed before 23.8 -> 22.5, 18.4 -> 17.5; but one layer again and
// again 9.7 -> 11.4, 7.6 -> 9.6, committed each time 19.8 -> 21.4, 16.9 -> 18.5, two in turn 10.2 -> 12.1, 7.8 -> 9.8, every
// one twice 24.0 -> 24.0, 18.8 -> 19.8 (1560 x 12 x 6 blocks: 42.9 -> 44.4), attention on it just before (those) 122.7 -> 123.8.
// What a read-back or a merge writes is what its caller reads next: never (read-back and a copy of it 23.8 us, 27.3 with
// streaming stores).
#pragma once
#include <atomic>
#include <cstdint>
#include <memory>
#include <new>

namespace ifx {

constexpr int64_t STREAM_FROM = (int64_t)300 << 20;
inline bool commit_streams(int64_t bytes_read_and_written) { return bytes_read_and_written > STREAM_FROM; }

// What a cache's calls have read of its layers.  A read-back streams where more than the line was moved since its layer was
// read last (by a read-back or by attention; a commit's blocks are found in the caches either way), and the
// read-backs go from layer to layer: the second of one layer is the sign that there may be a third.  A layer larger than the line
// streams always, and none where the caches can hold all.  Calls at once (attention's may be) find the counts of
// one order or another; what they decide is speed only.
class read_history {
  public:
    bool init(int layers)  // false: no host memory
    {
        read_at_.reset(new (std::nothrow) std::atomic<int64_t>[(size_t)layers]);
        if (!read_at_) return false;
        for (int l = 0; l < layers; ++l) read_at_[(size_t)l].store(LONG_AGO, std::memory_order_relaxed);
        return true;
    }
    // attention that reads `bytes` of a layer's blocks
    void attended(int layer, int64_t bytes) { (void)pass(layer, bytes); }
    // a read-back that moves `bytes`, of a cache whose layers hold as much that read-backs would move bytes_of_all: whether it streams
    bool read(int layer, int64_t bytes, int64_t bytes_of_all)
    {
        const int run = last_.exchange(layer, std::memory_order_relaxed) == layer ? 0 : run_.load(std::memory_order_relaxed) + 1;
        run_.store(run < 2 ? run : 2, std::memory_order_relaxed);
        const int64_t since = pass(layer, bytes);
        return bytes_of_all > STREAM_FROM && (bytes > STREAM_FROM || (run >= 2 && since > STREAM_FROM));
    }

  private:
    static constexpr int64_t LONG_AGO = -((int64_t)1 << 62);
    // bytes moved since the layer was read last, these included
    int64_t pass(int layer, int64_t bytes)
    {
        const int64_t now = moved_.fetch_add(bytes, std::memory_order_relaxed) + bytes;
        return now - read_at_[(size_t)layer].exchange(now, std::memory_order_relaxed);
    }
    std::unique_ptr<std::atomic<int64_t>[]> read_at_;  // what had been moved when the layer was read last
    std::atomic<int64_t> moved_{0};
    std::atomic<int> last_{-1}, run_{0};  // layer of the last read-back, and of how many layers in a row (2: or more)
};

}  // namespace ifx
