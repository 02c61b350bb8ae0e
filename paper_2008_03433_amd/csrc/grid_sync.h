// Waiting for the other workgroups inside a kernel whose workgroups are all resident at once.
#pragma once

#include "device_util.h"

namespace tron {

// A barrier over the grid costs a round trip to where every XCD sees the same memory for each step of its chain, and the
// additions to one counter, and the polls of it, go one after the other.  Up to kSyncFlat workgroups one counter does: 1.1 us with 40
// workgroups, 1.4 with 64, but 2.1 with 128 and 3.7 with 256.  Beyond, eight groups with a counter and a word to poll each,
// and a counter over the groups: 1.6 us with 128, 1.8 with 256 (sixteen groups: the same; a flag per workgroup, all of them
// polled by everyone: 4.1).  A launch that depends on the one before it costs 4 to 6 us.
constexpr int kSyncGroups = 8;
constexpr unsigned kSyncFlat = 64;
constexpr int kSyncLine = 32;   // 128 bytes apart
constexpr int kSyncWords = (3 + 2 * kSyncGroups) * kSyncLine;

// words: kSyncWords of device memory, zero between kernels (the workgroup that leaves last clears them)
struct GridSync {
    unsigned *words;
    long long ticks;   // how long a workgroup waits for the others (100 MHz); below zero: not at all
};

// Every thread of every workgroup makes the same calls.  What one workgroup reads of another's has to be written by store_shared before
// arrive() and read by load_shared after wait().  A workgroup that has waited for too long -- part of the grid is not
// resident -- gives up: wait() then returns false there and, soon, in every other workgroup; the caller leaves and the host takes
// another way.  So no wait is without an end, whatever else runs on the GPU.
class GridBarrier {
public:
    __device__ explicit GridBarrier(const GridSync &s) : w_(s.words), ticks_(s.ticks), round_(0) {}

    __device__ __forceinline__ void arrive()
    {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // every wavefront's own stores have arrived
        __syncthreads();
        ++round_;
        if (threadIdx.x != 0) return;
        const unsigned G = gridDim.x;
        if (G <= kSyncFlat) {
            add(root());
        } else {
            const unsigned g = blockIdx.x % kSyncGroups, members = (G - g + kSyncGroups - 1) / kSyncGroups;
            if (add(counter(g)) == round_ * members - 1 && add(root()) == round_ * kSyncGroups - 1)
                for (int k = 0; k < kSyncGroups; ++k) put(release(k), round_);
        }
    }

    __device__ __forceinline__ bool wait()
    {
        __shared__ int ok;
        if (threadIdx.x < kWave) {
            const bool flat = gridDim.x <= kSyncFlat;
            const unsigned *word = flat ? root() : release(blockIdx.x % kSyncGroups);
            const unsigned want = flat ? round_ * gridDim.x : round_;
            const bool good = poll(word, want);
            if (threadIdx.x == 0) {
                ok = good;
                if (!good) put(given_up(), 1u);
            }
        }
        __syncthreads();
        return ok;
    }

    // A lane waits until *place is no longer `empty`, adds what is there to sum and makes the place empty again.  False: given up, like
    // wait(); the workgroup must not arrive any more.
    __device__ __forceinline__ bool take(uint64_t *place, uint64_t empty, double &sum)
    {
        if (ticks_ >= 0) {
            const long long from = wall_clock64();
            for (unsigned polls = 1;; ++polls) {
                const uint64_t v = __hip_atomic_load(place, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (v != empty) {
                    sum += __longlong_as_double((long long)v);
                    __hip_atomic_store(place, empty, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    return true;
                }
                if ((polls & 15u) == 0 && (get(given_up()) != 0 || wall_clock64() - from > ticks_)) break;
            }
        }
        put(given_up(), 1u);
        return false;
    }

    // A wavefront waits until the first n words of every workgroup's line are no longer `empty` (a lane's own line, at most kWave
    // workgroups), and has them in v; 0 beyond.  False: given up, like wait().
    template <int N>
    __device__ __forceinline__ bool collect(const uint64_t *line, int n, uint64_t empty, double (&v)[N])
    {
        const bool mine = (threadIdx.x & (kWave - 1)) < gridDim.x;
        if (ticks_ >= 0) {
            const long long from = wall_clock64();
            for (unsigned polls = 1;; ++polls) {
                bool there = true;
#pragma unroll
                for (int k = 0; k < N; ++k) {
                    const uint64_t w = (mine && k < n) ? __hip_atomic_load(line + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
                    there &= w != empty;
                    v[k] = __longlong_as_double((long long)w);
                }
                if (__ballot(!there) == 0) return true;
                if ((polls & 15u) == 0 && (get(given_up()) != 0 || wall_clock64() - from > ticks_)) break;
            }
        } else {
#pragma unroll
            for (int k = 0; k < N; ++k) v[k] = 0.0;
        }
        if ((threadIdx.x & (kWave - 1)) == 0) put(given_up(), 1u);
        return false;
    }

    // the last thing a workgroup does, whether it gave up or not.  Every wavefront's additions and stores to the words have arrived before the
    // workgroup counts itself out: one still on its way (an addition whose result nobody waited for, given_up from take()) would
    // otherwise land behind the clearing and let the next launch's first barrier pass too early.
    __device__ __forceinline__ void leave()
    {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (threadIdx.x == 0 && add(left()) == gridDim.x - 1)
            for (int k = 0; k < kSyncWords / kSyncLine; ++k) put(w_ + k * kSyncLine, 0u);
    }

private:
    __device__ __forceinline__ bool poll(const unsigned *word, unsigned want)
    {
        if (ticks_ < 0) return false;
        const long long from = wall_clock64();
        for (unsigned polls = 1;; ++polls) {
            if ((int)(get(word) - want) >= 0) return true;
            if ((polls & 15u) == 0 && (get(given_up()) != 0 || wall_clock64() - from > ticks_)) return false;
        }
    }
    __device__ unsigned *root() const { return w_; }
    __device__ unsigned *left() const { return w_ + kSyncLine; }
    __device__ unsigned *given_up() const { return w_ + 2 * kSyncLine; }
    __device__ unsigned *counter(int g) const { return w_ + (3 + g) * kSyncLine; }
    __device__ unsigned *release(int g) const { return w_ + (3 + kSyncGroups + g) * kSyncLine; }
    __device__ static unsigned add(unsigned *p) { return __hip_atomic_fetch_add(p, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
    __device__ static unsigned get(const unsigned *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
    __device__ static void put(unsigned *p, unsigned v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

    unsigned *w_;
    long long ticks_;
    unsigned round_;
};

}  // namespace tron
