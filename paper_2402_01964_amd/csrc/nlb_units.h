// nlb_units.h -- feature rows of any width read in units of U elements (one
// 16-byte load each) that never leave the row.  Private to libnlb.so.
//
// Unit c (c a multiple of U) stands for columns c .. c + U - 1 of a row of
// `dim` >= U elements.  The unit that the width cuts is read from the row's
// end backwards, columns dim - U .. dim - 1: its first unit_shared() elements
// are columns of the unit before and are not used, the others are the row's
// last columns.  So are units wholly past the width, with every element
// unused.  The weights of a cut unit are staged to match (unit_shift).  Plain
// integer arithmetic, the same in host and device code, so that a host build
// checks what the kernels compile.
#pragma once

#include <stdint.h>

#if defined(__HIPCC__)
#define NLB_UNITS_HD __host__ __device__ __forceinline__
#else
#define NLB_UNITS_HD inline
#endif

// First column that unit c is read from.
NLB_UNITS_HD uint32_t unit_start(uint32_t c, uint32_t dim, uint32_t U) { return c < dim - U ? c : dim - U; }

// Elements at the start of unit c (c < dim) that belong to the unit before.
NLB_UNITS_HD uint32_t unit_shared(uint32_t c, uint32_t dim, uint32_t U) { return c - unit_start(c, dim, U); }

// Whether some unit is cut.
NLB_UNITS_HD bool unit_cut(uint32_t dim, uint32_t U) { return dim % U != 0; }

// The weights of the unit that the width cuts, moved in place from column
// order (row[c + i] the weight of column c + i) to the order in which the unit
// is read; the unused elements get weight zero.
template <uint32_t U, typename T>
NLB_UNITS_HD void unit_shift(T *row, uint32_t dim) {
    const uint32_t have = dim % U, c = dim - have, t = U - have;
    T v[U];
#pragma unroll
    for (uint32_t i = 0; i < U; i++) v[i] = row[c + i];
#pragma unroll
    for (uint32_t i = 0; i < U; i++) {
        T x = (T)0.0f;
#pragma unroll
        for (uint32_t j = 0; j < U; j++)
            if (j < have && j + t == i) x = v[j];
        row[c + i] = x;
    }
}
