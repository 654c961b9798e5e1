// Choice of a side stream (no HIP in here: the device calls come in as functions).
#pragma once
#include <vector>

namespace vie {

// Keeps in `side`, which holds a stream, the first of up to `most` streams that
// runs beside the main one.  make(&s): whether a further stream could be made;
// beside(s): 1 it does, 0 it does not, -1 no answer; drop(s) destroys one.
// Where none is found, or the search cannot go on, the stream that was there
// stays: it serves, only without the overlap.  Returns whether one was found.
template <class Stream, class Make, class Drop, class Beside>
bool pick_side(Stream &side, int most, Make make, Drop drop, Beside beside) {
  std::vector<Stream> tried{side};
  bool found = false;
  for (;;) {
    const int r = beside(tried.back());
    if (r > 0) found = true;
    if (r != 0 || (int)tried.size() >= most) break;
    Stream next;
    if (!make(&next)) break;
    tried.push_back(next);
  }
  if (found) side = tried.back();
  for (const Stream &s : tried)
    if (s != side) drop(s);
  return found;
}

}  // namespace vie
