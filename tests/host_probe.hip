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

// words per lane and workgroups of the bit-sliced TAC kernel for a graph of C classes and R recvs, B samples: as launched
extern "C" int host_tac_sliced(int32_t C, int32_t R, int32_t B)
{
    Dag d;
    d.C = C; d.R = R; d.W = (R + 63) / 64; d.CW = (C + 63) / 64; d.CWpad = (d.CW + 15) / 16 * 16; d.N = C;
    d.sliced_made = true;
    d.d_colbits = reinterpret_cast<uint64_t *>(&d);             // (only its being there is looked at)
    TacArgs a{};
    a.B = B;
    int32_t *flags = nullptr;
    const int e = (int)launch_tac_sliced(d, a, (size_t)B * 4, (size_t)B * 4, &flags, nullptr);
    (void)hipFree(d.d_work);
    return e;
}
