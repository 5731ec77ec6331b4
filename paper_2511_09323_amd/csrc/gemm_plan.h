// Arithmetic shared by the matrix-core kernels and their launchers that depends on sizes only: plain C++, so that it can be
// checked on a CPU at sizes no test would allocate.
#pragma once

#if defined(__HIPCC__)
#define MOC_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define MOC_HOST_DEVICE inline
#endif

namespace moc {

// Offset of the last readable k row of a slice of `bk` rows in a k-major operand, `left` >= 1 rows before the end of the
// contraction: the k-row offsets of a slice are clamped to it.  The rows are clamped before the product is formed: left * ld does not
// fit 32 bits for contractions over a few hundred thousand tokens, bk * ld does (checked on the host).
MOC_HOST_DEVICE int last_row_offset(int left, int bk, int ld) { return ((left < bk ? left : bk) - 1) * ld; }

}  // namespace moc
