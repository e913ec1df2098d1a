// The sweep launchers of libamrmg on the brick tables of a built context, for
// tests/test_gpu_first_sweeps_pinned.py: the first two sweeps of a cycle in one
// launch, and the same two as separate launches.  All arrays are the caller's,
// sized for the whole hierarchy (512 values a brick; ffs 96).
#include "amrmg_state.hpp"

template <class T>
static void fused(amrmg_ctx *c, int b0, int nb, void *e, const void *r, double *ffs, int faces, int nt)
{
    launch_hgs_first2<T>(c->st, c->ds.M, b0, nb, (T *)e, (const T *)r, ffs, faces != 0, nt);
}

// (mode bits: 1 input is zero, 16 fine sums of the result)
template <class T>
static void separate(amrmg_ctx *c, int b0, int nb, void *e, void *tmp, const void *r, double *ffs, double *scrap,
                     int faces, int nt)
{
    launch_hgs<T>(c->st, c->ds.M, b0, nb, nullptr, (T *)tmp, (const T *)r, nullptr, nullptr, scrap, 1 | 16, nt);
    launch_hgs<T>(c->st, c->ds.M, b0, nb, (const T *)tmp, (T *)e, (const T *)r, nullptr, nullptr, ffs,
                  faces ? 16 : 0, nt);
}

extern "C" void shim_fused(amrmg_ctx *c, int f32, int b0, int nb, void *e, const void *r, double *ffs, int faces,
                           int nt)
{
    if (f32) fused<float>(c, b0, nb, e, r, ffs, faces, nt);
    else fused<double>(c, b0, nb, e, r, ffs, faces, nt);
}

extern "C" void shim_separate(amrmg_ctx *c, int f32, int b0, int nb, void *e, void *tmp, const void *r, double *ffs,
                              double *scrap, int faces, int nt)
{
    if (f32) separate<float>(c, b0, nb, e, tmp, r, ffs, scrap, faces, nt);
    else separate<double>(c, b0, nb, e, tmp, r, ffs, scrap, faces, nt);
}
