// The words that the control kernels post checks to (Post, kernels_ctl.hpp), as the host keeps and
// reads them: (call tag << 40) | (done << 32) | checks completed, one word per instance or 1D signal.
#pragma once
#include <cstddef>
#include <cstring>

namespace ffcz {

struct PostWords {
  unsigned long long* p = nullptr;  // n words, memory that the device writes too
  size_t n = 0;
  unsigned long long tag = 0;

  // A new call on the first `words` words: the next tag, and the words cleared.  Clearing them is
  // what keeps the words of earlier calls out of this one (a tag has 24 bits, and a word that only
  // large batches use can stand for any number of calls); the tag keeps out what the passes of a
  // call that failed may still post.
  void begin(size_t words) {
    tag = tag == 0xffffff ? 1 : tag + 1;
    memset(p, 0, words * sizeof(*p));
  }

  // Checks that this call has posted for word i (0: none yet), and whether its loop has ended.
  struct Seen {
    int checks;
    bool done;
  };
  Seen read(size_t i) const {
    const unsigned long long v = __atomic_load_n(p + i, __ATOMIC_RELAXED);
    if ((v >> 40) != tag) return Seen{0, false};
    return Seen{(int)(v & 0xffffffffu), ((v >> 32) & 1) != 0};
  }
};

}  // namespace ffcz
