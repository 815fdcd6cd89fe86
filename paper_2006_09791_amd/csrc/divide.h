// Divisions by reciprocals, and the byte offset that buffer accesses drop.  Host and device, without a header of HIP: a test
// checks the arithmetic with the host's compiler.
#pragma once

#ifdef __HIP__
#define GSPC_HD __attribute__((host, device, always_inline)) inline
#else
#define GSPC_HD inline
#endif

namespace gspc {

// n / d with mul = div_magic(d) = floor((2^32 - 1) / d): exact while (n + 1) * d <= 2^32, and at most one too low for any
// larger n below 2^32 - 1.  Without a special case for d = 1: its branch (or select) stood in every kernel's index arithmetic
// before the first load.
GSPC_HD unsigned fast_div(unsigned n, unsigned mul) { return (unsigned)((unsigned long long)(n + 1) * mul >> 32); }

// The same for all n below 2^32 - 1.
GSPC_HD unsigned fast_div_any(unsigned n, unsigned d, unsigned mul) {
    const unsigned q = fast_div(n, mul);
    return n - q * d >= d ? q + 1 : q;
}

inline unsigned div_magic(unsigned d) { return 0xffffffffu / d; }

// Buffer accesses out of range return zero or are dropped by the hardware, so invalid lanes are given this byte offset instead
// of being branched around.  (Only the lane's own offset counts for that: the scalar offset of the instruction is excluded
// from the check, so an access that may not happen needs this in the lane's.)
constexpr unsigned kOob = 0xffffff00u;

}  // namespace gspc
