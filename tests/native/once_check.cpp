// Host check of build_once (csrc/qpg_internal.hpp): a build that throws leaves nothing behind, a later call
// builds anew, and one that succeeded is kept.
#include <cstdio>
#include <stdexcept>

#include "qpg_internal.hpp"

struct Thing {
  static int alive;
  int part = 0;
  Thing() { ++alive; }
  ~Thing() { --alive; }
};
int Thing::alive = 0;

#define CHECK(x)                        \
  do {                                  \
    if (!(x)) {                         \
      std::printf("failed: %s\n", #x);  \
      return 1;                         \
    }                                   \
  } while (0)

int main() {
  Thing* slot = nullptr;
  int destroyed = 0, built = 0;
  auto call = [&](bool fail) {
    return qpg::build_once(
        slot,
        [&](Thing* t) {
          ++built;
          t->part = 1;
          if (fail) throw std::runtime_error("no memory");
          t->part = 2;
        },
        [&](Thing* t) {
          ++destroyed;
          delete t;
        });
  };
  for (int k = 1; k <= 2; ++k) {
    bool thrown = false;
    try {
      call(true);
    } catch (const std::runtime_error&) {
      thrown = true;
    }
    CHECK(thrown && slot == nullptr && destroyed == k && built == k && Thing::alive == 0);
  }
  Thing* t = call(false);
  CHECK(t == slot && t->part == 2 && built == 3 && Thing::alive == 1);
  CHECK(call(true) == t && built == 3 && destroyed == 2);
  delete slot;
  return 0;
}
