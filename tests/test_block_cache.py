"""The cache of device blocks against a driver of a stated size, on the CPU: kept
blocks never take the memory that the runtime and other allocators need,
blocks are reused, and every block goes back where it came from."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <string>
#include <vector>
#include "block_cache.h"

static const size_t GB = (size_t)1 << 30, MB = (size_t)1 << 20;

struct Card {                       // two devices of 288 GB
    size_t free_[2] = {288 * GB, 288 * GB};
    int dev = 0;
    std::map<void*, std::pair<int, size_t>> held;
    uintptr_t next = 4096;
    int mallocs = 0;
};
struct Fake {
    Card* c = nullptr;
    int device() { return c->dev; }
    bool alloc(void** p, size_t bytes, bool* oom) {
        *oom = bytes > c->free_[c->dev];
        if (*oom) return false;
        c->free_[c->dev] -= bytes;
        *p = (void*)(c->next += 4096);
        c->held[*p] = {c->dev, bytes};
        ++c->mallocs;
        return true;
    }
    bool free(void* p) {
        auto it = c->held.find(p);
        if (it == c->held.end()) { printf("freed a block that is not held\n"); exit(1); }
        c->free_[it->second.first] += it->second.second;
        c->held.erase(it);
        return true;
    }
    void sync() {}
    bool free_bytes(size_t* f) { *f = c->free_[c->dev]; return true; }
};
using Cache = hmx::BlockCache<Fake>;

#define EXPECT(x) do { if (!(x)) { printf("%s:%d: %s\n", name, __LINE__, #x); return 1; } } while (0)

struct Block { void* p; size_t n; };
static Block take(Cache& c, size_t n, bool* ok = nullptr) {
    Block b{nullptr, Cache::round(n)};
    bool oom, got = c.alloc(&b.p, &b.n, &oom);
    if (ok) *ok = got;
    return b;
}

// whenever blocks are kept, the floor is free
static bool reserved(Card& k, Cache& c) { return c.cached() == 0 || k.free_[k.dev] >= Cache::kFloor; }

// three FP64 handles of 45 GB, each build with a scratch of 60 GB, released, then
// builds of other sizes: the floor is free after each step, and the reserve once the
// handles' blocks have been passed over
static int sequence(const char* name) {
    Card k;
    Cache c(Fake{&k});
    std::vector<Block> live;
    for (int i = 0; i < 3; ++i) {
        Block s = take(c, 60 * GB), a = take(c, 30 * GB), b = take(c, 15 * GB);
        EXPECT(reserved(k, c));
        c.free(s.p, s.n);
        EXPECT(reserved(k, c));
        live.push_back(a);
        live.push_back(b);
    }
    for (auto& b : live) { c.free(b.p, b.n); EXPECT(reserved(k, c)); }
    live.clear();
    unsigned r = 12345;
    for (int i = 0; i < 20000; ++i) {
        r = r * 1664525u + 1013904223u;
        const size_t n = (size_t)((r >> 8) % 40000 + 1) * (i % 3 ? MB : MB / 1024);
        if (live.size() > 12 || (r >> 5) % 2) {
            if (!live.empty()) {
                const size_t q = (r >> 9) % live.size();
                c.free(live[q].p, live[q].n);
                live.erase(live.begin() + q);
            }
        } else {
            bool ok;
            Block b = take(c, n, &ok);
            EXPECT(ok);
            EXPECT(b.n >= n && b.n / 4 * 3 <= Cache::round(n));
            live.push_back(b);
        }
        // (blocks under kLarge come back without a look: MBs, of which few)
        EXPECT(c.cached() == 0 || k.free_[0] + 64 * MB >= Cache::kFloor);
    }
    return 0;
}

// a program that moves on from a full card to blocks of a few GB: the reserve is free
// after some hundred allocations, whatever the program's own passes leave
static int reserve(const char* name) {
    Card k;
    Cache c(Fake{&k});
    std::vector<Block> v;
    for (size_t n : {45, 45, 45, 60, 50, 30, 8}) v.push_back(take(c, n * GB));
    v.push_back(take(c, 5 * GB - 300 * MB));
    for (auto& b : v) c.free(b.p, b.n);
    EXPECT(k.free_[0] == 300 * MB && c.cached() == 288 * GB - 300 * MB);  // all of one pass
    for (int i = 0; i < 320; ++i) {
        Block t = take(c, 3 * GB + (i % 3) * MB * 64);
        c.free(t.p, t.n);
        EXPECT(reserved(k, c));
    }
    EXPECT(k.free_[0] >= Cache::kReserve && k.free_[0] < 80 * GB);
    return 0;
}

// a program whose own blocks leave 0.33 GB: its passes map nothing more
static int tight(const char* name) {
    Card k;
    Cache c(Fake{&k});
    k.free_[0] -= 5 * GB;
    const size_t n[5] = {110 * GB, 76 * GB, 80 * GB, 12 * GB, 5 * GB - 340 * MB};
    for (int pass = 0; pass < 5; ++pass) {
        Block b[5];
        for (int q = 0; q < 5; ++q) b[q] = take(c, n[q]);
        for (int q = 0; q < 5; ++q) c.free(b[q].p, b[q].n);
        EXPECT(k.mallocs == 5 && reserved(k, c));
    }
    return 0;
}

// a block of the same size is reused; a second build of the same sizes maps nothing
static int reuse(const char* name) {
    Card k;
    Cache c(Fake{&k});
    for (int i = 0; i < 4; ++i) {
        Block s = take(c, 60 * GB), a = take(c, 45 * GB), t = take(c, 1000);
        if (i) EXPECT(k.mallocs == 3);
        c.free(s.p, s.n); c.free(a.p, a.n); c.free(t.p, t.n);
    }
    EXPECT(c.fresh_bytes() == (int64_t)(105 * GB + 1024) && c.flushes() == 0);
    return 0;
}

// another allocator of the process takes memory: the next large block that comes
// back makes room, by the smallest recent block that covers what is missing
static int others(const char* name) {
    Card k;
    Cache c(Fake{&k});
    Block a = take(c, 100 * GB), b = take(c, 10 * GB), d = take(c, 20 * GB);
    c.free(b.p, b.n);
    c.free(a.p, a.n);
    k.free_[0] -= 158 * GB - 100 * MB;  // 0.1 GB left
    c.free(d.p, d.n);
    EXPECT(k.free_[0] == 10 * GB + 100 * MB && c.cached() == 120 * GB && k.held.count(b.p) == 0);
    return 0;
}

// but first by a block that the program has passed over for hundreds of allocations
static int old_first(const char* name) {
    Card k;
    Cache c(Fake{&k});
    Block a = take(c, 100 * GB), d = take(c, 20 * GB);
    c.free(a.p, a.n);
    for (int i = 0; i < 400; ++i) {
        c.free(d.p, d.n);
        d = take(c, 20 * GB);
    }
    k.free_[0] = 1 * GB;
    c.free(d.p, d.n);
    EXPECT(k.free_[0] == 101 * GB && k.held.count(d.p) && !k.held.count(a.p));
    return 0;
}

// a program that moves on to other sizes on a card full of idle blocks: after its first
// pass it keeps its own blocks and maps nothing more
static int moves_on(const char* name) {
    Card k;
    Cache c(Fake{&k});
    std::vector<Block> v;
    for (size_t n : {45, 45, 45, 60, 30, 20, 15, 10, 8, 5}) v.push_back(take(c, n * GB));
    for (auto& b : v) c.free(b.p, b.n);
    int m = 0;
    for (int pass = 0; pass < 6; ++pass) {
        Block s = take(c, 115 * GB), f = take(c, 12 * GB), u = take(c, 13 * GB), w = take(c, 25 * GB);
        c.free(f.p, f.n);
        c.free(s.p, s.n);
        Block x = take(c, 33 * GB);
        for (Block* b : {&u, &w, &x}) c.free(b->p, b->n);
        if (pass == 1) m = k.mallocs;
    }
    EXPECT(k.mallocs == m);
    return 0;
}

// builds of four kinds of handles, as allocated: scratch, factors, two pools, near
// field, with sizes that vary from input to input; three inputs of the last kind in
// turn map nothing more after the second round
struct Handle { Block b[3]; };
static Handle build(Cache& c, double scratch, double factors, double pool, double near) {
    Block small[40];
    for (auto& b : small) b = take(c, 1000);
    for (auto& b : small) c.free(b.p, b.n);
    auto sz = [](double g) { return (size_t)(g * (double)GB); };
    Block s = take(c, sz(scratch)), f = take(c, sz(factors));
    c.free(s.p, s.n);
    Handle h;
    h.b[0] = take(c, sz(pool));
    h.b[1] = take(c, sz(pool));
    c.free(f.p, f.n);
    h.b[2] = take(c, sz(near));
    return h;
}
static void close(Cache& c, Handle& h) { for (auto& b : h.b) c.free(b.p, b.n); }

static int rounds(const char* name) {
    for (unsigned seed = 1; seed <= 200; ++seed) {
        Card k;
        Cache c(Fake{&k});
        unsigned r = seed * 2654435761u;
        auto vary = [&] { r = r * 1664525u + 1013904223u; return 0.95 + 0.1 * (double)(r >> 8) / (1 << 24); };
        const double kinds[4][4] = {{82, 14.5, 7.3, 34.5}, {21, 4.2, 2.1, 7.4}, {77, 15, 15, 25}, {12, 2.3, 1.2, 8}};
        for (auto& d : kinds) {
            std::vector<Handle> v;
            for (int i = 0; i < 3; ++i) {
                const double j = vary();
                v.push_back(build(c, d[0] * j, d[1] * j, d[2] * j, d[3] * (0.8 + 0.2 * vary())));
            }
            for (int i = 0; i < 5; ++i) {
                const double j = vary();
                Handle h = build(c, d[0] * j, d[1] * j, d[2] * j, d[3] * (0.8 + 0.2 * vary()));
                close(c, h);
                if (i == 0) { close(c, v[2]); close(c, v[1]); }
            }
            close(c, v[0]);
        }
        double j[3] = {vary(), vary(), vary()}, n[3] = {vary(), vary(), vary()};
        int m = 0;
        for (int i = 0; i < 24; ++i) {
            if (i == 6) m = k.mallocs;
            Handle h = build(c, 92 * j[i % 3], 14.8 * j[i % 3], 7.4 * j[i % 3], 39 * (0.8 + 0.2 * n[i % 3]));
            close(c, h);
            EXPECT(reserved(k, c));
        }
        EXPECT(k.mallocs == m);
    }
    return 0;
}

// a request beyond the card fails, with everything idle given back and live blocks kept
static int too_large(const char* name) {
    Card k;
    Cache c(Fake{&k});
    Block a = take(c, 100 * GB), b = take(c, 50 * GB);
    c.free(b.p, b.n);
    bool ok;
    take(c, 200 * GB, &ok);
    EXPECT(!ok && c.cached() == 0 && k.held.size() == 1 && k.held.count(a.p));
    take(c, 188 * GB, &ok);  // all that is left: live data may use the reserve
    EXPECT(ok);
    return 0;
}

// blocks of another device are neither handed out nor given back for this one
static int devices(const char* name) {
    Card k;
    Cache c(Fake{&k});
    k.dev = 1;
    Block a = take(c, 100 * GB);
    c.free(a.p, a.n);
    k.dev = 0;
    Block b = take(c, 100 * GB), d = take(c, 188 * GB - 100 * MB);
    EXPECT(b.p != a.p && k.held.count(a.p) && c.cached() == 100 * GB);
    c.free(d.p, d.n);  // 0.1 GB was left: goes back at once
    EXPECT(k.held.count(a.p) && k.held.size() == 2 && c.cached() == 100 * GB);
    EXPECT(c.trim() == (int64_t)(100 * GB) && k.held.size() == 1 && k.held.count(b.p));
    return 0;
}

// a pointer of another allocator never enters
static int foreign(const char* name) {
    Card k;
    Cache c(Fake{&k});
    int x;
    c.free(&x, GB);
    EXPECT(c.cached() == 0);
    return 0;
}

// the work space of a repeated sort out of the cache, whose blocks are up to a third
// larger than asked: each buffer holds what the count needs, whatever the other does
static int sort_space(const char* name) {
    struct Buf { void* p = nullptr; size_t bytes = 0; };
    for (size_t more = 0; more <= 33; ++more) {
        Card k;
        Cache c(Fake{&k});
        const size_t n0 = 1000000;
        Block big = take(c, n0 * 8 * (100 + more) / 100);  // what an earlier build left
        c.free(big.p, big.n);
        hmx::SortSpace<Buf> s;
        auto grow = [&](Buf& b, size_t bytes) {
            if (b.p) c.free(b.p, b.bytes);
            Block got = take(c, bytes);
            b.p = got.p;
            b.bytes = got.n;
        };
        for (size_t n = n0; n < n0 * 2; n += n0 / 50) {
            const size_t keys = n * 8, scratch = n * 12 + n / 10;
            s.reserve(keys, scratch, grow);
            EXPECT(s.keys.bytes >= keys);
            EXPECT(s.scratch.bytes >= scratch);
        }
    }
    return 0;
}

int main(int argc, char** argv) {
    const std::string n = argv[1];
    if (n == "sequence") return sequence(argv[1]);
    if (n == "reuse") return reuse(argv[1]);
    if (n == "reserve") return reserve(argv[1]);
    if (n == "tight") return tight(argv[1]);
    if (n == "others") return others(argv[1]);
    if (n == "old_first") return old_first(argv[1]);
    if (n == "moves_on") return moves_on(argv[1]);
    if (n == "rounds") return rounds(argv[1]);
    if (n == "too_large") return too_large(argv[1]);
    if (n == "devices") return devices(argv[1]);
    if (n == "foreign") return foreign(argv[1]);
    if (n == "sort_space") return sort_space(argv[1]);
    return 2;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("block_cache")
    (d / "t.cpp").write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-pthread", "-I",
                           os.path.join(ROOT, "paper_1708_09707_amd", "csrc"), str(d / "t.cpp"),
                           "-o", str(d / "t")])
    return str(d / "t")


@pytest.mark.parametrize("case", ["sequence", "reuse", "reserve", "tight", "others", "too_large",
                                  "devices", "foreign", "old_first", "moves_on", "rounds",
                                  "sort_space"])
def test_block_cache(program, case):
    r = subprocess.run([program, case], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
