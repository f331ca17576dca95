// Host-side check of how launches over samples of mixed sizes are cut (compiled
// for the host only): every chunk of a segment longer than a chunk starts in
// exactly one window of the launch and no window finds anything else.
#include <cstdio>
#include <map>
#include <random>
#include <vector>

#include "../../paper_2608_23786_amd/csrc/lbm_device.h"

using namespace mclbm;

int main() {
  std::mt19937 rng(7);
  const int chunk = 1024;
  for (int trial = 0; trial < 400; ++trial) {
    const int nseg = 1 + int(rng() % 40);
    std::vector<Seg> segs(nseg);
    std::map<int, int> want;
    int total = 0;
    for (int s = 0; s < nseg; ++s) {
      // 2 to 64 k blocks, powers of two as n^3 / block is; some ensembles of small samples only
      const int blocks = 2 << (trial % 3 == 0 ? rng() % 10 : rng() % 16);
      segs[s] = Seg{s, total, blocks, 0};
      if (blocks > chunk)
        for (int k = 0; k < blocks; k += chunk) want[total + k] = 0;
      total += blocks;
    }
    for (int w = 0; w * chunk < total; ++w) {
      const BlockChunk c = chunk_in_window(segs.data(), nseg, total, chunk, w);
      if (c.count == 0) continue;
      const auto it = want.find(c.first);
      if (c.count != chunk || it == want.end() || it->second++ != 0) {
        std::fprintf(stderr, "trial %d window %d: chunk at %d of %d\n", trial, w, c.first, c.count);
        return 1;
      }
    }
    for (const auto& k : want)
      if (k.second != 1) {
        std::fprintf(stderr, "trial %d: chunk at %d not found\n", trial, k.first);
        return 1;
      }
  }
  std::printf("groups ok\n");
  return 0;
}
