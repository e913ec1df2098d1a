// Device buffers without room (paper_1812_03689_amd/csrc/amrmg_state.hpp) on
// a device of a fixed number of bytes, played by the functions below: a buffer
// that finds no room gets that of the particle records, of every context of
// the call, only inside a call, and not of records that a capture holds.
// Built and run by tests/test_spare_buffers.py.
#include <cstdio>
#include <cstdlib>
#include <map>

#include "amrmg_state.hpp"

static std::map<void *, size_t> live;
static size_t used, room = 1 << 20;
static int syncs;

extern "C" hipError_t hipMalloc(void **p, size_t n)
{
    if (used + n > room) return hipErrorOutOfMemory;
    *p = std::malloc(n);
    live[*p] = n;
    used += n;
    return hipSuccess;
}
extern "C" hipError_t hipFree(void *p)
{
    used -= live.at(p);
    live.erase(p);
    std::free(p);
    return hipSuccess;
}
extern "C" hipError_t hipGetLastError() { return hipSuccess; }
extern "C" hipError_t hipStreamSynchronize(hipStream_t)
{
    ++syncs;
    return hipSuccess;
}
extern "C" hipError_t hipHostFree(void *) { return hipSuccess; }
extern "C" hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }

static void need(bool ok, const char *m)
{
    if (ok) return;
    std::printf("spare buffers: %s\n", m);
    std::exit(1);
}

int main()
{
    {
        amrmg_ctx a, b;
        amrmg_ctx *both[2] = {&a, &b}, *one = &a;
        auto records = [](amrmg_ctx &c) {
            need(c.rec_own.ensure(300000) == hipSuccess, "records find room");
            c.rec = (double4 *)c.rec_own.p;
        };
        records(a);
        records(b);
        DBuf w;
        need(w.ensure(400000) == hipErrorOutOfMemory && a.rec && b.rec, "outside a call nothing is given back");
        {
            SpareRecords s(&one);
            need(w.ensure(400000) == hipSuccess && !a.rec && !a.rec_own.p && b.rec, "the call's context gives back");
        }
        need(syncs == 1, "after what was queued");
        w.release();
        records(a);
        a.rec_held = true;
        {
            SpareRecords s(&one);
            need(w.ensure(400000) == hipErrorOutOfMemory && a.rec, "records that a capture holds stay");
        }
        a.rec_held = false;
        {
            SpareRecords s(both, 2);
            {
                SpareRecords inner(&one);
                need(w.ensure(400000) == hipSuccess && !a.rec && b.rec, "a call inside a call: its own context");
            }
            w.release();
            need(w.ensure(700000) == hipSuccess && !b.rec, "every context of a batch");
            need(a.rec_own.ensure(300000) == hipErrorOutOfMemory, "nothing left to give back");
        }
        need(Spare::current() == nullptr, "none left behind");
    }
    need(used == 0 && live.empty(), "everything freed");
    std::printf("spare buffers ok\n");
    return 0;
}
