// Exchange slots of the resident tridiagonalisation (trd.hip): where the
// work-groups of a team publish y = A v and the next column of column c of a
// matrix of order n.  Offsets in doubles from the start of the matrix's
// exchange area; entry i of y at slot + 2 i, of the next column at slot +
// trd_slot_next(n) + 2 i, (re, im).
#pragma once

#include <stddef.h>

#if defined(__HIPCC__)
#define ZK_HD __host__ __device__ inline
#else
#define ZK_HD inline
#endif

namespace zk {

ZK_HD size_t trd_slot(int n, int c) { return 4 * (size_t)n * (size_t)c; }
ZK_HD size_t trd_slot_next(int n) { return 2 * (size_t)n; }
// columns 0 .. n-2 are exchanged: at most 4 n^2 doubles
ZK_HD size_t trd_slot_doubles(int n) { return 4 * (size_t)n * (size_t)(n - 1); }

}  // namespace zk
