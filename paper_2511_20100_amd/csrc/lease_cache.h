// A bounded cache of items that host threads hold while they enqueue device work, and that queued work still uses when they
// have let go of them.  Host code only.
#pragma once

#include <iterator>
#include <list>
#include <utility>

namespace mtmc {

// Item: movable; idle() = no queued work uses it any more, wait() returns once that is so.  Every call, and the destructor,
// is made under the owner's lock (only leases' holders use an entry's item outside of it).
//
// An entry that makes room for another leaves the cache at once and is destroyed when its last holder has released it and
// its work has ended: looked at on every insertion, and waited for only while more than `capacity` such entries are
// left, so that the memory is bounded and nobody waits for work that is not that entry's.
template <class Key, class Item>
class LeaseCache {
 public:
  struct Entry {
    Key key;
    Item item;
    int holders;
  };
  explicit LeaseCache(size_t capacity) : capacity_(capacity) {}
  LeaseCache(const LeaseCache&) = delete;
  LeaseCache& operator=(const LeaseCache&) = delete;
  ~LeaseCache() {
    for (Entry& e : live_) e.item.wait();
    for (Entry& e : retired_) e.item.wait();
  }

  // The entry of `key`, held, or nullptr.  It becomes the last one to make room.
  Entry* acquire(const Key& key) {
    for (auto it = live_.begin(); it != live_.end(); ++it)
      if (it->key == key) {
        live_.splice(live_.end(), live_, it);
        ++live_.back().holders;
        return &live_.back();
      }
    return nullptr;
  }
  // A new entry, held.
  Entry* insert(Key key, Item item) {
    live_.push_back(Entry{std::move(key), std::move(item), 1});
    if (live_.size() > capacity_) retired_.splice(retired_.end(), live_, live_.begin());
    for (auto it = retired_.begin(); it != retired_.end();) {
      auto next = std::next(it);
      if (it->holders == 0 && it->item.idle()) retired_.erase(it);
      it = next;
    }
    for (auto it = retired_.begin(); retired_.size() > capacity_ && it != retired_.end();) {
      auto next = std::next(it);
      if (it->holders == 0) {
        it->item.wait();
        retired_.erase(it);
      }
      it = next;
    }
    return &live_.back();
  }
  void release(Entry* e) { --e->holders; }

  size_t live() const { return live_.size(); }
  size_t retired() const { return retired_.size(); }

 private:
  size_t capacity_;
  std::list<Entry> live_;     // the one used longest ago first
  std::list<Entry> retired_;  // the one replaced first first
};

}  // namespace mtmc
