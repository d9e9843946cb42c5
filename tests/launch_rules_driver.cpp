// The launch rules of csrc/launch_rules.h as C functions, for test_launch_rules.py.
#include "launch_rules.h"

extern "C" {
int64_t serve_blocks(int64_t items, int parts) { return vr::serve_blocks(items, parts); }
void serve_part(int64_t block, int parts, int64_t *item, int *part) {
  const vr::ServePart p = vr::serve_part_of(block, parts);
  *item = p.item;
  *part = p.part;
}
}
