// Compute units handed from launch to launch (host code, no HIP calls).
//
// Launches whose workgroups wait for each other must find room for all of
// them, so the launches that can run at the same time must not want more
// compute units than there are.  Every unit belongs to the launch that took
// it last: a later launch that takes some of them is first ordered behind that
// launch, whether or not it has started, and then holds them itself.  Launches
// that are not ordered behind each other thus hold different units, whatever
// they were ordered behind before, and those of a launch are on loan until a
// later one takes them: at most as many shares are kept as there are units.
#pragma once
#include <cstddef>
#include <vector>

template <typename Stream, typename Event> class SwCuPool {
  public:
    explicit SwCuPool(int cus) : free_(cus) { shares_.reserve((size_t)cus + 1); }   // (never grown: a share has a unit)

    // Takes `want` units (at most all there are) for a launch on `stream`: those of launches before it on the stream
    // (behind which it is anyway), then free ones, then those of other launches, oldest first.  wait(event) orders the
    // stream behind a launch whose units are taken; false if that failed, and nothing is taken.
    template <typename Wait, typename Drop> bool take(int want, Stream stream, Wait wait, Drop drop) {
        int need = want;
        auto from = [&](bool same) {
            for (Share &s : shares_) {
                if ((s.stream == stream) != same) continue;
                s.taken = need < s.cus ? need : s.cus;
                need -= s.taken;
            }
        };
        from(true);
        const int idle = need < free_ ? need : free_;
        need -= idle;
        from(false);
        if (need > 0) return false;
        for (const Share &s : shares_)
            if (s.taken > 0 && !wait(s.event)) return false;
        free_ -= idle;
        size_t kept = 0;
        for (Share s : shares_) {
            s.cus -= s.taken;
            if (s.cus > 0) shares_[kept++] = s;
            else drop(s.event);
        }
        shares_.erase(shares_.begin() + kept, shares_.end());
        return true;
    }
    // The units taken are the launch's that `event` is recorded behind (or free, where there is none).
    void lend(int cus, Stream stream, Event event) { shares_.push_back(Share{event, stream, cus, 0}); }
    void put_back(int cus) { free_ += cus; }
    size_t shares() const { return shares_.size(); }

  private:
    struct Share {
        Event event;
        Stream stream;
        int cus, taken;   // units held; of those, taken by the launch at hand
    };
    std::vector<Share> shares_;   // oldest first
    int free_;
};
