"""The bookkeeping of kept scratch (csrc/scratch.h), on the host over a runtime that only counts: streams finish their
work when they are told to, the device has a fixed amount of memory, and its pool keeps what is freed to it."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2202_06088_amd", "csrc")

SRC = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <vector>
#include "scratch.h"
using namespace neuvv;

#define CHECK(x) do { if (!(x)) { printf("line %d: %s\n", __LINE__, #x); exit(1); } } while (0)

// Streams are numbers; work on one is a count, finished up to done[stream]. Waiting makes a stream depend on another's
// count. A block's last work is checked against what the next user waits for.
struct Ev { int stream = -1; long at = 0; };
struct Device {
    std::map<int, long> issued, done;
    std::map<int, std::map<int, long>> seen;   // stream -> work of other streams that it waits for
    std::map<char*, size_t> live;              // allocated, not freed
    std::map<char*, Ev> last;                  // the block's last use
    size_t used = 0, pooled = 0, room = (size_t)4 << 30;   // in use, free in the pool
    int allocs = 0, queries = 0, syncs = 0, events = 0;
    char* next = (char*)0x1000;
    // whether work of e is before anything that stream s does from now on
    bool ordered(const Ev& e, int s) {
        return e.stream < 0 || e.stream == s || done[e.stream] >= e.at || seen[s][e.stream] >= e.at;
    }
};
struct Rt {
    using Status = int;
    using Stream = int;
    using Event = Ev*;
    static constexpr int ok = 0;
    Device* d;
    int alloc(void** p, size_t bytes, int s) {
        const size_t reused = d->pooled >= bytes ? bytes : 0;   // (a larger one needs memory of its own)
        if (d->used + d->pooled - reused + bytes > d->room) return 2;
        ++d->allocs;
        d->pooled -= reused;
        d->used += bytes;
        *p = d->next;
        d->live[d->next] = bytes;
        d->next += bytes;
        return 0;
    }
    static bool no_memory(int e) { return e == 2; }
    int free(void* p, int s) {
        CHECK(d->live.count((char*)p));
        CHECK(d->ordered(d->last[(char*)p], s));
        d->used -= d->live[(char*)p];
        d->pooled += d->live[(char*)p];
        d->live.erase((char*)p);
        return 0;
    }
    int create(Ev** e) { ++d->events; *e = new Ev; return 0; }
    void destroy(Ev* e) { --d->events; delete e; }
    int record(Ev* e, int s) { e->stream = s; e->at = d->issued[s]; return 0; }
    int wait(int s, Ev* e) { long& v = d->seen[s][e->stream]; if (v < e->at) v = e->at; return 0; }
    bool passed(Ev* e) { ++d->queries; return d->done[e->stream] >= e->at; }
    int finish(int s) { d->done[s] = d->issued[s]; return 0; }
    int trim() { d->pooled = 0; return 0; }
    int sync(Ev* e) { ++d->syncs; long& v = d->done[e->stream]; if (v < e->at) v = e->at; return 0; }
};

// One call: a block (kept or from the pool), some work on it, given back.
struct Call { void* p; size_t bytes; int stream; };
static Call begin(KeptScratch<Rt>& k, Rt& rt, size_t bytes, int s) {
    Call c{nullptr, bytes, s};
    if (k.acquire(rt, &c.p, bytes, s) != 0) c.p = nullptr;
    if (c.p) {
        CHECK(rt.d->live[(char*)c.p] >= bytes);
        CHECK(rt.d->ordered(rt.d->last[(char*)c.p], s));   // nothing else may still use it
    } else {
        CHECK(rt.alloc(&c.p, bytes, s) == 0);
    }
    rt.d->last[(char*)c.p] = Ev{s, ++rt.d->issued[s]};
    return c;
}
static void end(KeptScratch<Rt>& k, Rt& rt, const Call& c) {
    rt.d->last[(char*)c.p] = Ev{c.stream, ++rt.d->issued[c.stream]};
    int st = 0;
    if (!k.put_back(rt, c.p, c.stream, &st)) CHECK(rt.free(c.p, c.stream) == 0);
}
static void call(KeptScratch<Rt>& k, Rt& rt, size_t bytes, int s) { end(k, rt, begin(k, rt, bytes, s)); }
static void finish(Device& d, int s) { d.done[s] = d.issued[s]; }

static const size_t KiB = 1024, MiB = 1024 * KiB;

int main(int argc, char** argv) {
    Device d;
    Rt rt{&d};
    auto* kp = new KeptScratch<Rt>;
    KeptScratch<Rt>& k = *kp;
    const char* what = argv[1];
    if (!strcmp(what, "size")) {   // blocks are close to what was asked for; larger requests are not kept
        for (size_t b : {1 * KiB, 64 * KiB, 65 * KiB, 1 * MiB, MiB + 1, 32 * MiB + 5, 33 * MiB, 63 * MiB + 1, 64 * MiB})
            CHECK(k.block_bytes(b) >= b && (b <= 64 * KiB || k.block_bytes(b) < (b <= MiB ? 2 * b : b + 2 * MiB)));
        call(k, rt, 33 * MiB, 1);
        CHECK(k.bytes() == 34 * MiB);
        call(k, rt, 64 * MiB + 1, 2);
        CHECK(k.blocks() == 1);
    } else if (!strcmp(what, "streams")) {   // eight streams' smallest adjoints are kept side by side
        for (int r = 0; r < 5; ++r)
            for (int s = 0; s < 8; ++s) call(k, rt, 33 * MiB, s);
        CHECK(d.allocs == 8 && k.bytes() == 8 * 34 * MiB);
    } else if (!strcmp(what, "dropped")) {   // streams come and go: their blocks serve the next ones
        for (int s = 0; s < 200; ++s) {
            call(k, rt, 100 * KiB, s);
            call(k, rt, 33 * MiB, s);
            finish(d, s);
        }
        CHECK(k.blocks() <= k.kBlocks && k.bytes() <= k.kBytes);
        const int before = d.allocs;
        call(k, rt, 33 * MiB, 1000);
        CHECK(d.allocs == before);
        // but not while their work still runs
        for (int s = 2000; s < 2100; ++s) call(k, rt, 33 * MiB, s);
        CHECK(d.allocs > before + 80);
    } else if (!strcmp(what, "outgrown")) {   // a stream's needs grow: what it has outgrown goes back
        for (size_t b = 64 * KiB; b <= 64 * MiB; b *= 2) call(k, rt, b, 7);
        CHECK(k.blocks() == 1 && d.used == 64 * MiB);
        call(k, rt, 64 * KiB, 7);
        CHECK(k.blocks() == 1);
    } else if (!strcmp(what, "nested")) {   // a call that holds one block while it takes another settles on two
        for (int r = 0; r < 10; ++r) {
            Call a = begin(k, rt, 40 * MiB, 3), b = begin(k, rt, 300 * KiB, 3);
            CHECK(a.p != b.p);
            end(k, rt, b);
            end(k, rt, a);
        }
        CHECK(d.allocs == 2 && k.blocks() == 2);
    } else if (!strcmp(what, "memory")) {   // a device without room for a new block: the idle ones can be given back
        d.room = 60 * MiB;
        call(k, rt, 30 * MiB, 1);
        void* p = nullptr;
        CHECK(k.acquire(rt, &p, 40 * MiB, 2) == 2 && !p);
        CHECK(k.give_back(rt, 2) == 0 && d.used == 0 && d.pooled == 0);
        CHECK(k.blocks() == 0 && k.bytes() == 0 && d.events == 0);
        CHECK(k.acquire(rt, &p, 40 * MiB, 2) == 0 && p);
        CHECK(k.give_back(rt, 2) == 0 && k.blocks() == 1);   // (held by a call: left alone)
        // a call that finds no memory takes back what is idle by itself, but not while its stream is captured
        int st = 0;
        CHECK(k.put_back(rt, p, 2, &st));
        CHECK(k.serve(rt, &p, 55 * MiB, 3, true, true) == 2);
        CHECK(k.serve(rt, &p, 55 * MiB, 3, true, false) == 0 && d.used == 56 * MiB);
        CHECK(k.put_back(rt, p, 3, &st));
        d.room = 57 * MiB;   // less than the block of this request would take
        CHECK(k.serve(rt, &p, 57 * MiB, 4, true, false) == 0 && d.used == 57 * MiB && !k.put_back(rt, p, 4, &st));
    } else {   // random calls on a few and on many streams, some overlapping on one stream, some finishing late
        srand(atoi(what));
        std::vector<Call> open;
        for (int i = 0; i < 20000; ++i) {
            const int s = rand() % (rand() % 2 ? 4 : 80);
            if (open.size() < 6 && rand() % 2) open.push_back(begin(k, rt, ((size_t)1 << (10 + rand() % 18)) + rand() % 5000, s));
            else if (!open.empty()) {
                const int j = rand() % open.size();
                end(k, rt, open[j]);
                open.erase(open.begin() + j);
            }
            if (rand() % 3 == 0) finish(d, rand() % 80);
            if (rand() % 4000 == 0) CHECK(k.release(rt, s) == 0);
            CHECK(k.blocks() <= k.kBlocks && k.bytes() <= k.kBytes && d.events == k.blocks());
            for (size_t a = 0; a < open.size(); ++a)
                for (size_t b = 0; b < a; ++b) CHECK(open[a].p != open[b].p);
        }
        for (auto& c : open) end(k, rt, c);
        CHECK(k.release(rt, 0) == 0 && d.used == 0);
    }
    printf("ok\n");
}
"""


@pytest.fixture(scope="module")
def keep(tmp_path_factory):
    d = tmp_path_factory.mktemp("keep")
    (d / "keep.cpp").write_text(SRC)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-I", CSRC, str(d / "keep.cpp"), "-o", str(d / "keep"), "-pthread"])
    return str(d / "keep")


@pytest.mark.parametrize("what", ["size", "streams", "dropped", "outgrown", "nested", "memory", "1", "2", "3", "4"])
def test_kept_scratch_bookkeeping(keep, what):
    r = subprocess.run([keep, what], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.endswith("ok\n"), r.stdout + r.stderr
