// The three streams of a cache: made for four caches at a time, and left to later caches when a cache is destroyed.
//
// The runtime ties a stream to one of its four hardware queues when the stream is made: to the one that has the fewest streams then, the
// last of those (as the queue ids in kernel traces show).  A side stream on the queue of its caller's stream runs the match behind the
// experts instead of beside them - four steps of rows of 5,120 over 2,000 traces take 580 us instead of 437 - and with streams made for each
// cache, the queue depends on all that the process has made and destroyed before: after caches of other models one cache in three had the
// caller's, or two, where the caller made streams of its own in between.  Beside the default stream alone, the side streams of four
// sets made in a row get the fourth, second, third and fourth queue, and that stream has the first.
#pragma once

#include <mutex>
#include <vector>

namespace moei {

template <typename Stream>
struct StreamSet {
    Stream prefetch{}, copy{}, side{};
    int device = -1;
    long made = -1;  // sets before this one in the process
};

constexpr int kSetsTogether = 4;

// At most kKept idle sets of a device; any thread.
template <typename Stream, int kKept>
class StreamSets {
    static_assert(kKept >= kSetsTogether, "the sets made besides are kept");

public:
    // The set of `device` that was made first, of those that `usable` accepts (a set that it refuses is forgotten: the device was reset);
    // where there is none, the first of kSetsTogether that `make` fills in, with its result (`drop`: for what a later one of them leaves
    // that cannot be made, which is no failure).
    template <typename Usable, typename Make, typename Drop>
    int take(int device, StreamSet<Stream>* out, Usable usable, Make make, Drop drop) {
        std::lock_guard<std::mutex> lock(mutex_);
        for (;;) {
            int first = -1;
            for (int i = 0; i < (int)idle_.size(); ++i)
                if (idle_[i].device == device && (first < 0 || idle_[i].made < idle_[first].made)) first = i;
            if (first < 0) break;
            *out = idle_[first];
            idle_.erase(idle_.begin() + first);
            if (usable(*out)) return 0;
        }
        auto next = [&](StreamSet<Stream>* s) {
            *s = StreamSet<Stream>{};
            s->device = device;
            s->made = made_++;
            return make(s);
        };
        const int rc = next(out);
        for (int i = 1; i < kSetsTogether && rc == 0; ++i) {
            StreamSet<Stream> more;
            if (next(&more) != 0 || !put(more)) {
                drop(more);
                break;
            }
        }
        return rc;
    }
    // False: there is no room, the set remains the caller's.
    bool keep(const StreamSet<Stream>& s) {
        std::lock_guard<std::mutex> lock(mutex_);
        return put(s);
    }

private:
    bool put(const StreamSet<Stream>& s) {
        int n = 0;
        for (const auto& i : idle_) n += i.device == s.device;
        if (n >= kKept) return false;
        try {
            idle_.push_back(s);
        } catch (...) {
            return false;
        }
        return true;
    }

    std::mutex mutex_;
    std::vector<StreamSet<Stream>> idle_;
    long made_ = 0;
};

}  // namespace moei
