// Which contracted element a GEMM stage's offset-table entry stands for
// (fno_gemm.hip); plain C++, so that the host can replay it.
#pragma once

namespace fno {

// Entry i of the offset table of a chunk of klen contracted elements.  The
// table covers whole stages; entries past the chunk repeat elements of its
// last quad, each at its own place in the quad: where an operand is read four
// elements at a time (klen a multiple of four then) a load past the chunk is a
// whole quad inside it again, aligned as every other.
constexpr int gemm_k_entry(int i, int klen) {
  if (i < klen) return i;
  const int e = ((klen - 1) & ~3) + (i & 3);
  return e < klen ? e : klen - 1;
}

}  // namespace fno
