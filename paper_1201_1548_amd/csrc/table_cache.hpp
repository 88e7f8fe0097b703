// Tables built on demand and kept for later calls, within a limit.
#pragma once
#include <stddef.h>
#include <stdint.h>

#include <algorithm>
#include <memory>
#include <mutex>
#include <utility>
#include <vector>

namespace bires {

// The tables of one kind.  A table of a tag serves the requests of that tag for
// at most its sizes (a, b).  A request that none serves builds one: large enough
// for the tag's present tables too where that stays below `one` bytes, so that
// requests that grow in turn leave one table and not a row of outgrown ones,
// which it replaces.  Above `all` bytes in total the least recently used tables
// go.  A table that goes is destroyed when its last holder lets it go: the
// calls in flight and the captured graphs hold the tables they read.
template <class Mem>
class TableCache {
 public:
  struct Table {
    int a = 0, b = 0;
    std::shared_ptr<Mem> mem;  // null: none
  };
  using Gone = std::vector<std::shared_ptr<Mem>>;

  TableCache(size_t one, size_t all) : one_(one), all_(all) {}

  // size(a, b): a table's bytes; build(a, b): the table, null on failure.  join:
  // build for the tag's present tables too.  gone receives the tables that went.
  template <class Size, class Build>
  Table get(int tag, int a, int b, bool join, Size size, Build build, Gone* gone) {
    std::lock_guard<std::mutex> lk(mu_);
    if (Entry* e = find(tag, a, b)) return use(*e);
    if (join) {
      int ja = a, jb = b;
      for (const Entry& e : v_)
        if (e.tag == tag) ja = std::max(ja, e.t.a), jb = std::max(jb, e.t.b);
      if (size(ja, jb) <= one_) a = ja, b = jb;
    }
    Entry n;
    n.tag = tag;
    n.t.a = a;
    n.t.b = b;
    n.bytes = size(a, b);
    if (n.bytes > one_ || n.bytes > all_) return Table();
    n.t.mem = build(a, b);
    if (!n.t.mem) return Table();
    drop([&](const Entry& e) { return e.tag == tag && e.t.a <= a && e.t.b <= b; }, gone);
    while (!v_.empty() && total() + n.bytes > all_) {
      uint64_t oldest = v_[0].used;
      for (const Entry& e : v_) oldest = std::min(oldest, e.used);
      drop([&](const Entry& e) { return e.used == oldest; }, gone);
    }
    v_.push_back(std::move(n));
    return use(v_.back());
  }

  // The same if a table serves it already.
  Table look(int tag, int a, int b) {
    std::lock_guard<std::mutex> lk(mu_);
    Entry* e = find(tag, a, b);
    return e ? use(*e) : Table();
  }

  void clear(Gone* gone) {
    std::lock_guard<std::mutex> lk(mu_);
    drop([](const Entry&) { return true; }, gone);
  }

  size_t bytes() {
    std::lock_guard<std::mutex> lk(mu_);
    return total();
  }

 private:
  struct Entry {
    int tag = 0;
    Table t;
    size_t bytes = 0;
    uint64_t used = 0;
  };

  Entry* find(int tag, int a, int b) {
    Entry* hit = nullptr;
    for (Entry& e : v_)
      if (e.tag == tag && e.t.a >= a && e.t.b >= b && (!hit || e.bytes < hit->bytes)) hit = &e;
    return hit;
  }
  Table use(Entry& e) {
    e.used = ++clock_;
    return e.t;
  }
  size_t total() const {
    size_t s = 0;
    for (const Entry& e : v_) s += e.bytes;
    return s;
  }
  template <class Pred>
  void drop(Pred p, Gone* gone) {
    for (size_t i = 0; i < v_.size();) {
      if (!p(v_[i])) {
        ++i;
        continue;
      }
      gone->push_back(std::move(v_[i].t.mem));
      v_.erase(v_.begin() + i);
    }
  }

  const size_t one_, all_;
  std::mutex mu_;
  std::vector<Entry> v_;
  uint64_t clock_ = 0;
};

}  // namespace bires
