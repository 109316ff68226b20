// Copies from device memory to pageable host memory in parallel pieces.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>

namespace iblbm {

struct HostCopy {
  void *dev;
  void *host;
  size_t bytes;
};

// Copies every piece to the host and returns when all are done.  The device
// memory must be idle (the stream that wrote it has been synchronised).  Runs on
// the current device.
//
// A plain hipMemcpy to pageable memory goes through one staging buffer by one
// thread, which also takes the page faults of a freshly allocated array: 10
// GB/s (32.9 ms for the fields of 7175 x 2014 nodes, 347 MB; 3.7 ms for 2000 x
// 800).  Here a few threads each move blocks through a pinned buffer of their
// own, so that one's copy and faults overlap the others' transfers (9.3 and 1.5
// ms).  The other way a plain copy reaches 28 GB/s and stays.  Copies below 4
// MB, into memory that is not pageable, and while another thread has the buffers
// are plain ones.
hipError_t host_copy(const HostCopy *pieces, int n);

// Sims and servers share the pinned buffers (12 MB, made at the first large
// copy); the last one to go gives them back.
void host_copy_retain();
void host_copy_release();

}  // namespace iblbm
