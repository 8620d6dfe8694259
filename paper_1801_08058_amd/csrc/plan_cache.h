// Per-thread cache of launch plans (host code).
//
// Planning a launch (kernel selection, strip / tile geometry, split of a reduction) is a pure function of the
// descriptor, a few integers and the environment switches.  The planning functions keep what they computed per thread,
// keyed by their arguments, so that the second call with a descriptor costs a few table look-ups instead of the
// geometry loops; ngc_reload_switches() invalidates everything.
#pragma once
#include <string.h>

#include <unordered_map>

#include "common.h"

namespace ngc {

// Key: plain 32-bit words without padding, compared and hashed as such
template <class Key>
struct PlanKeyHash {
    size_t operator()(const Key &k) const
    {
        static_assert(sizeof(Key) % 4 == 0, "hashed as words");
        const uint32_t *w = reinterpret_cast<const uint32_t *>(&k);
        uint64_t h = 0xcbf29ce484222325ull;
        for (size_t i = 0; i < sizeof(Key) / 4; ++i) h = (h ^ w[i]) * 0x100000001b3ull;
        return (size_t)(h ^ (h >> 29));
    }
};
template <class Key>
struct PlanKeyEq {
    bool operator()(const Key &x, const Key &y) const { return memcmp(&x, &y, sizeof(Key)) == 0; }
};

template <class Key, class V>
struct KeyedPlanCache {
    std::unordered_map<Key, V, PlanKeyHash<Key>, PlanKeyEq<Key>> map;
    uint32_t epoch = 0xFFFFFFFFu;
    V *find(const Key &k)
    {
        if (epoch != sw_epoch()) {
            map.clear();
            epoch = sw_epoch();
        }
        auto it = map.find(k);
        return it == map.end() ? nullptr : &it->second;
    }
    V &put(const Key &k, const V &v)
    {
        if (map.size() >= 2048) map.clear();             // a process cycling through more nodes than that replans
        return map[k] = v;
    }
};

}  // namespace ngc
