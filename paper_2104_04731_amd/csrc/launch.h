// Host side of a launch: the kernel launch itself, and small per-thread tables of plans.
#pragma once
#include <hip/hip_runtime.h>

#include <string.h>

#include <tuple>
#include <utility>

namespace c2i8 {

// hipLaunchKernel itself, its status returned: 2.4 us of host time where <<<>>> followed by hipGetLastError takes
// 2.6-2.9 (3000 empty kernels back to back).  A refused launch leaves no error behind for the caller's next check.
template <typename A>
hipError_t launch(void (*kern)(A), dim3 grid, dim3 block, size_t lds, hipStream_t st, const A &a)
{
    void *args[] = {const_cast<void *>(static_cast<const void *>(&a))};
    const hipError_t e = hipLaunchKernel(reinterpret_cast<const void *>(kern), grid, block, args, lds, st);
    if (e != hipSuccess) (void)hipGetLastError();
    return e;
}

template <typename... P, typename... A, size_t... I>
hipError_t launch_values(void (*kern)(P...), dim3 grid, dim3 block, size_t lds, hipStream_t st, std::index_sequence<I...>, A &&...a)
{
    std::tuple<P...> values{static_cast<P>(a)...};
    void *args[] = {static_cast<void *>(const_cast<std::remove_const_t<P> *>(&std::get<I>(values)))...};
    const hipError_t e = hipLaunchKernel(reinterpret_cast<const void *>(kern), grid, block, args, lds, st);
    if (e != hipSuccess) (void)hipGetLastError();
    return e;
}
template <typename P0, typename P1, typename... P, typename... A>
hipError_t launch(void (*kern)(P0, P1, P...), dim3 grid, dim3 block, size_t lds, hipStream_t st, A &&...a)
{
    static_assert(sizeof...(A) == 2 + sizeof...(P), "one value per kernel argument");
    return launch_values(kern, grid, block, lds, st, std::index_sequence_for<P0, P1, P...>{}, std::forward<A>(a)...);
}

// Table of up to N plans.  A network calls the same layers over and over, and choosing how one runs costs the host 4.5 us
// in the middle, 11 at the 95th percentile (1233 one-shot, NHWC and dilated calls), with kept weights 7.9 and 15.7 (267): the
// tile model 2.7, the resident kernel's candidates 2.3 (kept weights: 2.8), the stream kernel's 0.6 to 2.9 -- against the 2.4 us of a launch.  These were taken before the panel kernel, whose
// eight tiles with up to six pixel counts each add 0.6 to 0.8 us in the middle on another host (4000 layers of 65 to 512 channels for each kind of call, all new: 9.2 to
// 10.1 -> 9.9 to 10.8; of 16 to 512 channels 0.4 to 0.7).  A problem is looked for from its hash's slot on, up to
// the first empty one, so N problems never displace one another (two of 20 would meet in a direct-mapped table of 64 with a
// probability of 95 %, and evict each other on every call); in a full table a new one replaces the plan at its hash's
// slot.  Key: plain integers without padding, compared whole.  Meant to be thread_local: no locks, bounded, and gone with
// the thread.
template <typename Key, typename Val, int N>
class PlanTable {
    static_assert((N & (N - 1)) == 0, "a power of two");
    struct Entry {
        Key key;
        Val val;
    };
    unsigned hash_[N] = {};   // 0: empty
    Entry e_[N] = {};

public:
    // The plan of `key`, made by fill(&val) on a miss (fill returns false: nothing to keep, null comes back).  It stays where
    // it is until the next call.
    template <typename F>
    const Val *get(const Key &key, F &&fill)
    {
        unsigned h = 2166136261u;
        const unsigned char *b = reinterpret_cast<const unsigned char *>(&key);
        for (size_t i = 0; i + 4 <= sizeof(Key); i += 4) {
            unsigned w;
            memcpy(&w, b + i, 4);
            h = (h ^ w) * 2654435761u;
            h ^= h >> 15;
        }
        const unsigned first = h & (N - 1);
        h |= 0x80000000u;
        unsigned at = first;
        for (int i = 0; i < N && hash_[at]; ++i, at = (at + 1) & (N - 1))
            if (hash_[at] == h && memcmp(&e_[at].key, &key, sizeof(Key)) == 0) return &e_[at].val;
        Val made{};
        if (!fill(&made)) return nullptr;
        e_[at].key = key;   // an empty slot, or, all N taken, the first one again
        e_[at].val = made;
        hash_[at] = h;
        return &e_[at].val;
    }
};

}  // namespace c2i8
