// Checks gwc::kernels_may_use on every kind of pointer (CPU only).
#include <cstdio>

#include "gwc_pointers.h"

int main() {
  int bad = 0;
  for (int device = 0; device < 2; ++device)
    for (int managed = 0; managed < 2; ++managed)
      for (int owner = -1; owner < 3; ++owner)
        for (int current = 0; current < 3; ++current) {
          gwc::PointerKind k;
          k.device = device;
          k.managed = managed;
          k.owner = owner;
          const bool want = device && !managed && owner == current;
          if (gwc::kernels_may_use(k, current) != want) {
            std::printf("device %d managed %d owner %d current %d\n", device, managed, owner, current);
            ++bad;
          }
        }
  if (!bad) std::printf("all checks passed\n");
  return bad != 0;
}
