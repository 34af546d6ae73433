// What a test of the library's host side says to the stand-in for the HIP runtime (host_runtime.cpp).
#pragma once
#include <cstdint>

extern "C" {
void host_fail_launch(const char *kernel, int after);   // of the launches whose name holds `kernel`, the one after `after` others fails
void host_fail_malloc(int after);                       // the hipMalloc after `after` others
void host_set_last_error(int e);                        // the calling thread's last error, as a failed call before left it
void host_malloc_takes(int ms);                         // each hipMalloc, from now on
int64_t host_malloc_bytes();                            // by hipMalloc so far
int host_event_records();                               // hipEventRecord calls so far
int64_t host_copied_bytes();                            // brought from pinned buffers so far, by whichever kernel
int host_launches(const char *kernel);                  // launches so far whose name holds `kernel`
}
