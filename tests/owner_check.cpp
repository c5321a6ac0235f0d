// Host-only check of stream_owner (paper_2502_06155_amd/csrc/tile_attn_host.cpp), linked against
// the built library and run by tests/test_stream_owner.py: hipStreamPerThread is a stream of
// its own in every thread, so each thread gets a number there that no other one has, also
// after it has ended; every other handle is the same stream in all threads (0).
#include <cstdio>
#include <set>
#include <thread>
#include <vector>

#include "host_internal.h"

int main() {
  using ta::host::stream_owner;
  void* per_thread = (void*)2;  // hipStreamPerThread
  std::set<uint64_t> seen;
  for (int round = 0; round < 3; ++round) {  // threads of later rounds may reuse ended ones' ids
    std::vector<uint64_t> got(8), again(8), other(8);
    std::vector<std::thread> threads;
    for (int i = 0; i < 8; ++i)
      threads.emplace_back([&, i] {
        got[i] = stream_owner(per_thread);
        again[i] = stream_owner(per_thread);
        other[i] = stream_owner(nullptr) + stream_owner((void*)0x1000);
      });
    for (auto& t : threads) t.join();
    for (int i = 0; i < 8; ++i)
      if (got[i] == 0 || got[i] != again[i] || other[i] != 0 || !seen.insert(got[i]).second)
        return std::printf("thread %d of round %d: %llu\n", i, round, (unsigned long long)got[i]), 1;
  }
  std::printf("stream owners ok\n");
  return 0;
}
