// Device memory of resident indexes, kept for a while after an index is freed.
//
// The driver clears memory before it hands it out again, at about 38 GB/s on
// MI355X: a program that opens one reference after the other soon waits for
// that (16 Mbp, whose index takes 4.6 GB: 122 ms per index from the fiftieth
// on, against 6 ms for everything else).  Blocks of freed indexes are
// therefore kept for the next one: at most kKeepBytes per device, and no more
// than a quarter of what is free besides (asked for every kKeepFreely: the
// question takes 5 us), given back when they have not been used for
// kKeepSeconds, when an allocation of the library finds too little memory,
// or when dev_trim is called.
#pragma once

#include <hip/hip_runtime.h>
#include <cstddef>
#include <initializer_list>

namespace samatch {

constexpr size_t kKeepBytes = (size_t)8 << 30;
constexpr size_t kKeepFreely = (size_t)512 << 20;
constexpr int kKeepSeconds = 2;

// Memory on the current device, at least 256-byte aligned, contents undefined.
hipError_t dev_alloc(void **p, size_t bytes);

// hipMalloc for everything else the library allocates: when there is too
// little memory, what is kept is given back and it is tried again.
hipError_t dev_malloc(void **p, size_t bytes);

// Returns blocks of dev_alloc on one device (NULL: none).  Waits for all work
// on it first, as hipFree does, so that no kernel uses a block that another
// index has taken.
void dev_free(std::initializer_list<void *> ps);

// Bytes kept on a device (free as far as a caller of dev_alloc is concerned).
size_t dev_kept(int device);

// Gives everything kept on a device back; the bytes that were.
size_t dev_trim(int device);

}  // namespace samatch
