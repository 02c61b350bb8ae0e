// Host-side helpers of dataset creation.
#pragma once

#include <algorithm>
#include <exception>
#include <memory>
#include <thread>
#include <vector>

namespace tron {

// An array whose elements start undefined: where every element is written by the threads that fill it, clearing it first (as
// std::vector does) would touch every page once more, on one thread.
template <typename T>
class HostArray {
public:
    explicit HostArray(size_t n = 0) : p_(n ? new T[n] : nullptr) {}
    T *data() const { return p_.get(); }
    T &operator[](size_t i) const { return p_[i]; }

private:
    std::unique_ptr<T[]> p_;
};

// threads for `work` entries of a pass: at most eight, and at least some 64 thousand entries each (starting a thread takes some
// tens of microseconds)
inline unsigned host_threads(int64_t work)
{
    const unsigned most = std::max(1u, std::min(8u, std::thread::hardware_concurrency()));
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>(most, work >> 16));
}

// fn(t, T) for t = 0 .. T - 1, on T threads if they can be had.  fn must not throw.
template <class F>
void on_threads(unsigned T, F &&fn)
{
    std::vector<std::thread> workers;
    unsigned started = 1;
    try {
        for (; started < T; ++started) workers.emplace_back(fn, started, T);
    } catch (const std::exception &) {
        // no more threads to be had: the remaining shares run below
    }
    fn(0u, T);
    for (unsigned t = started; t < T; ++t) fn(t, T);
    for (std::thread &w : workers) w.join();
}

// fn(first, last) over [0, n) cut into equal ranges, one thread per range; work = entries the whole pass touches.  fn must not
// throw and must write only what belongs to its own range.
template <class F>
void parallel_ranges(int64_t n, int64_t work, F &&fn)
{
    const unsigned T = host_threads(work);
    const int64_t per = (n + T - 1) / T;
    on_threads(T, [&](unsigned t, unsigned) { fn(std::min<int64_t>(n, (int64_t)t * per), std::min<int64_t>(n, (int64_t)(t + 1) * per)); });
}

}  // namespace tron
