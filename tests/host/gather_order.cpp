// Host check of which tile order the gathers of sem_ax take (test
// infrastructure): arguments nx ny nz N bytes-per-word, output "tiles chunked".
// Compiled for the host with hipcc by tests/test_gather_order.py.
#include <cstdio>
#include <cstdlib>

#include "sem_types.h"

using namespace semk;

int main(int argc, char **argv) {
  if (argc != 6) return 2;
  const Box b = Box::make(atoi(argv[1]), atoi(argv[2]), atoi(argv[3]), atoi(argv[4]));
  const int word = atoi(argv[5]);
  const int64_t nt = upd_num_tiles(b, word == 8, kGatherShape);
  std::printf("%lld %d\n", (long long)nt, (int)gather_chunked(nt, b.L() * word, word == 8, false));
  return 0;
}
