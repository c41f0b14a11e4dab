// The choice of a library product's algorithm (host code, no HIP headers): a
// candidate may run only where the caller's workspace holds what it needs, and
// a choice that is kept must not be reused where it does not.
#pragma once

#include <cstddef>
#include <map>
#include <mutex>
#include <utility>

namespace pa {

// The first of n candidates (ok(i), need(i)) that runs in ws_bytes; -1: none.
template <typename Ok, typename Need>
int first_fit(int n, size_t ws_bytes, Ok&& ok, Need&& need) {
  for (int i = 0; i < n; ++i)
    if (ok(i) && need(i) <= ws_bytes) return i;
  return -1;
}

// Choices kept per problem.  Workspaces of about the same size (whole MiB)
// share a choice, so that a problem tuned with one workspace stays tuned with
// another; a call whose workspace is too small for the shared choice has one
// of its own, by its exact size.
template <typename Key, typename Algo>
class AlgoCache {
 public:
  bool find(const Key& key, size_t ws_bytes, Algo* algo) {
    std::lock_guard<std::mutex> lk(mu_);
    auto it = shared_.find({key, ws_bytes >> 20});
    if (it == shared_.end()) return false;
    if (it->second.need > ws_bytes) {
      it = exact_.find({key, ws_bytes});
      if (it == exact_.end()) return false;
    }
    *algo = it->second.algo;
    return true;
  }
  void keep(const Key& key, size_t ws_bytes, const Algo& algo, size_t need) {
    std::lock_guard<std::mutex> lk(mu_);
    auto it = shared_.find({key, ws_bytes >> 20});
    if (it != shared_.end() && it->second.need > ws_bytes)
      exact_[{key, ws_bytes}] = {algo, need};
    else
      shared_[{key, ws_bytes >> 20}] = {algo, need};
  }

 private:
  struct Entry {
    Algo algo;
    size_t need;
  };
  using Map = std::map<std::pair<Key, size_t>, Entry>;
  std::mutex mu_;
  Map shared_, exact_;
};

}  // namespace pa
