// pick_side (csrc/side.h) with made-up streams: numbers 0 (the one that is
// there), 1, 2, ...  Arguments: streams that can be made beside it, the most to
// try, then each stream's answer (1 runs beside, 0 does not, -1 none).
// Prints: found, the stream kept, streams made, streams dropped.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "side.h"

int main(int argc, char **argv) {
  const int can = std::atoi(argv[1]), most = std::atoi(argv[2]);
  std::vector<int> answer;
  for (int i = 3; i < argc; ++i) answer.push_back(std::atoi(argv[i]));
  int side = 0, made = 0;
  std::vector<int> dropped;
  const bool found = vie::pick_side(
      side, most,
      [&](int *s) {
        if (made == can) return false;
        *s = ++made;
        return true;
      },
      [&](int s) { dropped.push_back(s); }, [&](int s) { return answer.at(s); });
  std::printf("%d %d %d", (int)found, side, made);
  for (int s : dropped) std::printf(" %d", s);
  std::printf("\n");
  return 0;
}
