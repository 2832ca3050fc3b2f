// Calls into the library's launchers that no entry point reaches in a test (host_lib.py).
#include "internal.h"

using namespace tictac;

// the class grouping on the device for N compute ops with rows of W words (nothing is read or written)
extern "C" int host_group_rows(int32_t N, int32_t W)
{
    Dag d;
    d.N = N;
    d.W = W;
    return (int)launch_group_rows(d, nullptr, nullptr, nullptr);
}
extern "C" int64_t host_group_bytes(int32_t N) { return (int64_t)group_workspace_bytes(N); }
