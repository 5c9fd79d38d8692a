// Values worked out once per launch shape (a query of the runtime costs tens of
// microseconds) and shared by every context of the process, on whatever thread.
// Host code only, so that a plain C++ compiler takes it.
#pragma once

#include <map>
#include <mutex>

namespace pl {

template <class Key> class LaunchCache {
public:
    // The value of a key; make() works it out the first time.
    template <class Make> int get(const Key &key, Make make)
    {
        std::lock_guard<std::mutex> lock(mu_);
        const auto f = values_.find(key);
        if (f != values_.end()) return f->second;
        return values_[key] = make();
    }

private:
    std::mutex mu_;
    std::map<Key, int> values_;
};

}  // namespace pl
