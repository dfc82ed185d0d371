// kept.hpp -- what the library keeps of past calls, up to a number of entries
// and bytes; the entry unused for longest goes first.
#pragma once

#include <cstddef>
#include <cstdint>
#include <map>
#include <memory>
#include <utility>
#include <vector>

namespace spinqp {

// Not synchronised: callers hold their own lock, and let go of what insert
// returns outside it (destroying an entry may wait for the device).
template <typename V>
class Kept {
  public:
    using Key = std::vector<double>;
    Kept(size_t most, size_t most_bytes) : most_(most), most_bytes_(most_bytes) {}

    // The entry of `key`, or null.  pin: it stays until clear().
    std::shared_ptr<V> find(const Key& key, bool pin = false) {
        const auto it = map_.find(key);
        if (it == map_.end()) return nullptr;
        it->second.used = ++clock_;
        it->second.pinned |= pin;
        return it->second.value;
    }

    // Adds or replaces the entry of `key`; the entries that had to go.  An entry
    // larger than the bound alone is kept, by itself.
    std::vector<std::shared_ptr<V>> insert(const Key& key, std::shared_ptr<V> value, size_t bytes, bool pin = false) {
        std::vector<std::shared_ptr<V>> gone;
        const auto old = map_.find(key);
        if (old != map_.end()) {
            gone.push_back(std::move(old->second.value));
            pin |= old->second.pinned;
            bytes_ -= old->second.bytes;
            map_.erase(old);
        }
        map_[key] = Entry{std::move(value), bytes, ++clock_, pin};
        bytes_ += bytes;
        while (map_.size() > most_ || bytes_ > most_bytes_) {
            auto least = map_.end();
            for (auto it = map_.begin(); it != map_.end(); ++it)
                if (!it->second.pinned && it->second.used != clock_ &&
                    (least == map_.end() || it->second.used < least->second.used))
                    least = it;
            if (least == map_.end()) break;
            gone.push_back(std::move(least->second.value));
            bytes_ -= least->second.bytes;
            map_.erase(least);
        }
        return gone;
    }

    std::vector<std::shared_ptr<V>> clear() {
        std::vector<std::shared_ptr<V>> gone;
        for (auto& kv : map_) gone.push_back(std::move(kv.second.value));
        map_.clear();
        bytes_ = 0;
        return gone;
    }

    size_t size() const { return map_.size(); }
    size_t bytes() const { return bytes_; }

  private:
    struct Entry {
        std::shared_ptr<V> value;
        size_t bytes = 0;
        uint64_t used = 0;
        bool pinned = false;
    };
    size_t most_, most_bytes_, bytes_ = 0;
    uint64_t clock_ = 0;
    std::map<Key, Entry> map_;
};

}  // namespace spinqp
