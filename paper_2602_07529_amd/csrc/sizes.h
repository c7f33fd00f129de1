// Size arithmetic of the host code.
#pragma once
#include <stddef.h>
#include <stdint.h>

static inline int64_t dag_ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
static inline size_t dag_align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }
