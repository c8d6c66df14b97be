// Host buffers of a call outlive the stream that uses them, whichever way the
// call ends (streams.hpp, pinned.hpp over a stub of the runtime).
#include <cstdio>
#include <new>
#include <vector>

#include "pinned.hpp"
#include "streams.hpp"

using namespace tn;

static int bad = 0;
static void check(bool ok, const char* what) {
    if (!ok) {
        std::printf("BAD %s\n", what);
        bad = 1;
    }
}

static bool alive = false, alive_at_sync = false;
struct Buffer {  // a host image that says whether it is there
    Buffer() { alive = true; }
    ~Buffer() { alive = false; }
};

int main() {
    int s;
    stub_on_sync = [] { alive_at_sync = alive; };
    // an exception behind the first launch: drained while the image is there
    try {
        Buffer host;
        DrainGuard guard(&s);
        throw std::bad_alloc();
    } catch (const std::bad_alloc&) {
    }
    check(stub_syncs == 1 && alive_at_sync, "an exception drains before the buffers go");
    stub_syncs = 0;
    {
        Buffer host;
        DrainGuard guard(&s);
        guard.drained();
    }
    check(stub_syncs == 0, "a drained call does not wait again");
    // side streams first, then the caller's
    {
        Buffer host;
        DrainGuard guard(&s);
        SideStreams side(2);
        check(side.size() == 2, "side streams");
    }
    check(stub_syncs == 3, "side streams and the caller's are drained");

    // pinned blocks: the pool holds what was given back
    uint8_t* first;
    {
        PinnedBlock b(true);
        first = b.p;
        b.in_use(&s);
        b.drained();
    }
    stub_syncs = 0;
    {
        PinnedBlock b(true);
        check(b.p == first, "a drained block is used again");
        b.in_use(&s);
    }
    check(stub_syncs == 1, "a block in use is drained before it is given back");
    {
        PinnedBlock b(true);
        check(b.p == first, "and then used again");
        b.in_use(&s);
        stub_sync_result = hipErrorUnknown;
    }
    stub_sync_result = hipSuccess;
    {
        PinnedBlock b(true);
        check(b.p && b.p != first, "a block that could not be drained is not used again");
    }
    PinnedBlock none(false);
    check(!none.p, "no block unless wanted");
    if (!bad) std::printf("ok\n");
    return bad;
}
