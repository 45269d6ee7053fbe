// Contraction steps of the channel mix's weight gradient: host-compilable, so
// that the rule can be checked without a GPU.
//
// The contraction of degree l runs over batch x mcount columns (b, m), in steps
// of 16.  Member by member, a member's orders rounded up to whole steps, a lane
// loads its four consecutive orders by two vector loads; with all columns in one
// row it takes each by its own (member, order), which costs more a step.  The
// line lies where the one row saves a fifth of the steps.  Weight gradient by
// tiles, us, member by member / in one row: 64 x 64 channels, lmax 8: 155 / 60,
// 64 x 96, lmax 200 of 4 orders: 211 / 55, 32 x 128, lmax 24: 147 / 95.
#pragma once

namespace sht {
namespace mixm {

constexpr int kStep = 16;

constexpr int member_steps(int batch, int mcount) { return batch * ((mcount + kStep - 1) / kStep); }
constexpr int row_steps(int batch, int mcount) { return (batch * mcount + kStep - 1) / kStep; }
// 2^21: the kernel's float32 quotient column / mcount is exact below it; 2^32: a
// member's values (complex) as a 32-bit factor
constexpr bool one_row(int batch, int mcount, unsigned long long member) {
  return static_cast<long long>(batch) * mcount < (1 << 21) && member < (1ULL << 32) &&
         5LL * row_steps(batch, mcount) <= 4LL * member_steps(batch, mcount);
}
constexpr int steps(int batch, int mcount, unsigned long long member) {
  return one_row(batch, mcount, member) ? row_steps(batch, mcount) : member_steps(batch, mcount);
}
// member of a column
constexpr int member_of(int column, float one_over_mcount) {
  return static_cast<int>((static_cast<float>(column) + 0.5f) * one_over_mcount);
}

}  // namespace mixm
}  // namespace sht
