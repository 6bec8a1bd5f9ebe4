// Host-only test of what an autotune cache key holds
// (paper_2511_16298_amd/csrc/tunecache.hpp), built with sanitizers by
// tests/test_tune_key_cpu.py.  Takes a scratch directory; prints OK and exits 0
// when every check holds.
#include <stdio.h>

#include <string>

#include "tunecache.hpp"

using ss::TuneChoice;
using ss::TuneKey;

static int g_fail = 0;
#define CHECK(c)                                                            \
  do {                                                                      \
    if (!(c)) {                                                             \
      fprintf(stderr, "%s:%d: check failed: %s\n", __FILE__, __LINE__, #c); \
      ++g_fail;                                                             \
    }                                                                       \
  } while (0)

static TuneKey key(uint32_t spread, uint32_t flags) {
  TuneKey k;
  k.arch = "gfx950";
  k.runtime = 70226015;
  k.abi = 1;
  k.frames_log2 = 6;
  k.gaussians_log2 = 26;
  k.pairs_log2 = 28;
  k.tile_bits = 19;
  k.frame_tile_bits = 13;
  k.spread = spread;
  k.caller_flags = flags;
  return k;
}

int main(int argc, char** argv) {
  if (argc != 2) return 2;
  const std::string path = std::string(argv[1]) + "/tune.txt";
  TuneChoice c;
  // a choice recorded before the spread passes: the same sizes, not taken
  FILE* f = fopen(path.c_str(), "w");
  CHECK(f != nullptr);
  if (f == nullptr) return 1;
  fprintf(f, "ss-tune 1 gfx950 70226015 1 6 26 28 19 13 = 8 8 512 0 3.940000\n");
  fclose(f);
  CHECK(!ss::tune_cache_lookup(path.c_str(), key(1, 0), &c));
  CHECK(!ss::tune_cache_lookup(path.c_str(), key(0, 0), &c));
  // frames that the spread passes serve, frames they do not, other flags: an
  // entry each, and the old line stays
  CHECK(ss::tune_cache_store(path.c_str(), key(1, 0), TuneChoice{8, 16, 512, 0, 2.25}));
  CHECK(!ss::tune_cache_lookup(path.c_str(), key(0, 0), &c));
  CHECK(!ss::tune_cache_lookup(path.c_str(), key(1, 4), &c));
  CHECK(ss::tune_cache_store(path.c_str(), key(0, 0), TuneChoice{6, 8, 512, 0, 3.0}));
  CHECK(ss::tune_cache_store(path.c_str(), key(1, 4), TuneChoice{8, 8, 512, 0, 3.5}));
  CHECK(ss::tune_cache_lookup(path.c_str(), key(1, 0), &c) && c.radix_bits == 8 && c.items == 16);
  CHECK(ss::tune_cache_lookup(path.c_str(), key(0, 0), &c) && c.radix_bits == 6 && c.items == 8);
  CHECK(ss::tune_cache_lookup(path.c_str(), key(1, 4), &c) && c.items == 8);
  std::string text;
  f = fopen(path.c_str(), "r");
  CHECK(f != nullptr);
  for (int ch; f != nullptr && (ch = fgetc(f)) != EOF;) text.push_back(static_cast<char>(ch));
  if (f != nullptr) fclose(f);
  CHECK(text.find("ss-tune 1 gfx950 70226015 1 6 26 28 19 13 = 8 8 512 0 3.940000\n") == 0);
  if (g_fail == 0) printf("OK\n");
  return g_fail == 0 ? 0 : 1;
}
