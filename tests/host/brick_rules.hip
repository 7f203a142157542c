// Prints what the kernels per block shape (csrc/pbz_brick.h) decide on the host.  Reads lines from standard input:
//   "tiles wide compress array index pruned elements BW BZ BY BX": the values that a lane holds for such a call.
// Built for the host only; nothing here runs on a GPU.
#include <cstdio>
#include <iostream>
#include <string>

#include "pbz_brick.h"

int main() {
  std::string what;
  while (std::cin >> what) {
    if (what == "tiles") {
      int wide, compress, array, index, pruned, b[4];
      int64_t elements;
      std::cin >> wide >> compress >> array >> index >> pruned >> elements >> b[0] >> b[1] >> b[2] >> b[3];
      const pbz::brick::Tiles t = pbz::brick::tiles(wide != 0, compress != 0, array, index, pruned != 0, b[0], b[1], b[2], b[3]);
      std::printf("%d\n", elements <= t.few_to ? t.few : t.many);
    } else {
      return 1;
    }
  }
  return 0;
}
