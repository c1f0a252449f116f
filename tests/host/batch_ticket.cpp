// What the batch kernels are handed as their completion slot is no larger
// than the 256 bytes that a batch's workspace and each of a server's round
// slots keep for it.
#include <cstdint>
#include <cstdio>

#include "sel_device.h"

int main() {
  const sel::BatchArgs* b = nullptr;
  const sel::LutArgs* l = nullptr;
  if (sizeof(*b->slot) > 256 || sizeof(*l->slot) > 256) {
    std::printf("a batch's slot takes %zu and %zu bytes\n", sizeof(*b->slot), sizeof(*l->slot));
    return 1;
  }
  std::printf("ok\n");
  return 0;
}
