// How the workgroups of a tile share its finish out, without the memory behind it: the kernels run it on a word of device
// memory (MeetWord in device_util.hpp), a host test through every order of its steps.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ts {

// One thread of each workgroup calls this after its workgroup's partial sums are
// acknowledged.  Bits 0 - 7 of the word count arrivals, bit 8 + s says that workgroup s has left.  Returns the
// workgroups whose share the caller takes: its own once all have arrived, and for the last to arrive also those of workgroups that
// had left by then.  A workgroup without a share, or that has waited long enough, leaves: the
// others need not be resident, and no share is taken twice or not at all, because arriving and leaving are changes of one word.
// At most 16 workgroups.  The word is cleared before the next launch that uses it.
template <class Word>
__host__ __device__ __forceinline__ uint32_t meet_splits(Word &word, int expected, int self, bool share) {
  const uint32_t before = word.add(1);
  if ((int)(before & 255u) == expected - 1) return before >> 8 | 1u << self;
  if (!share) return 0;
  word.start_clock();
  for (;;) {
    uint32_t now = word.load();
    const bool late = word.late();
    if ((int)(now & 255u) != expected && late) now = word.set(256u << self);
    if ((int)(now & 255u) == expected) return 1u << self;
    if (late) return 0;
    word.nap();
  }
}

}  // namespace ts
