// The merged task lists (dag.hpp, launch_list) against a plain stable sort of all
// blocks' tasks by latest start level, earliest start level and block, with schedules
// shared between the lists and without.  Prints the number of lists.
#include <algorithm>
#include <cstdio>
#include <random>

#include "../../paper_2507_06938_amd/csrc/dag.hpp"

using namespace dl::dag;

static std::vector<uint64_t> sorted(const std::vector<int>& nbks, const std::vector<char>& inv,
                                    bool chain) {
  struct Key {
    int alap, asap;
    uint64_t word;
  };
  std::vector<Key> all;
  for (size_t b = 0; b < nbks.size(); ++b) {
    std::vector<Task> q;
    std::vector<int> asap, alap;
    levels(nbks[b], inv[b] != 0, chain, q, asap, alap);
    for (size_t t = 0; t < q.size(); ++t) all.push_back({alap[t], asap[t], pack(q[t], (int)b)});
  }
  std::stable_sort(all.begin(), all.end(), [](const Key& x, const Key& y) {
    return x.alap != y.alap ? x.alap < y.alap : x.asap < y.asap;
  });
  std::vector<uint64_t> out;
  for (const Key& k : all) out.push_back(k.word);
  return out;
}

int main() {
  std::mt19937 g(3);
  Schedules shared;
  int lists = 0;
  for (int it = 0; it < 300; ++it) {
    std::vector<int> nbks(1 + g() % 9);
    std::vector<char> inv(nbks.size());
    for (size_t b = 0; b < nbks.size(); ++b) {
      nbks[b] = b && g() % 3 == 0 ? nbks[b - 1] : 1 + (int)(g() % 20);
      inv[b] = (char)(g() % 2);
    }
    const bool chain = it % 4 != 0;
    const std::vector<uint64_t> want = sorted(nbks, inv, chain);
    if (launch_list(nbks, inv, chain) != want) return 1;
    if (launch_list(nbks, inv, chain, &shared) != want) return 2;
    ++lists;
  }
  // one schedule per size, inverse and chain, however many lists use it
  if (shared.all.size() > 20 * 2 * 2) return 3;
  std::printf("ok %d lists\n", lists);
  return 0;
}
