"""The pool of destroyed plans' memory (csrc/block_pool.h) on a stub device: what
is handed out again, the bounds, that memory running out anywhere in the
library gives the idle blocks back and tries again, and a wait that fails."""
import os
import subprocess

from paper_2503_18479_amd import build as B

PROGRAM = r"""
#include "block_pool.h"
#include <cassert>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <thread>
#include <vector>
static std::mutex mu;
static std::map<void *, size_t> live;   // what the stub device has handed out
static size_t used = 0, capacity = ~(size_t)0, waits = 0, big = 0;
static int wait_result = 0;
struct Dev {
    static constexpr int no_memory = 2;
    static int alloc(void **p, size_t n) {
        std::lock_guard<std::mutex> l(mu);
        if (n == 7) return 5;                       // fails for another reason
        if (used + n > capacity) return no_memory;
        *p = std::malloc(1);
        live[*p] = n;
        used += n;
        return 0;
    }
    static void free(void *p) {
        std::lock_guard<std::mutex> l(mu);
        assert(live.count(p));
        used -= live[p];
        live.erase(p);
        std::free(p);
    }
    static int wait() { std::lock_guard<std::mutex> l(mu); ++waits; return wait_result; }
};
typedef cosim::BlockPool<Dev> Pool;
static const size_t MB = 1 << 20;
int main() {
    void *p, *q;
    size_t n, m;
    {   // a block of the right size and device comes back, after a wait
        Pool pool;
        assert(pool.take(0, 10 * MB, &p, &n) == 0 && n >= 10 * MB && waits == 0);
        pool.give(0, p, n);
        assert(pool.take(1, 10 * MB, &q, &m) == 0 && q != p && waits == 0);   // another device
        pool.give(1, q, m);
        assert(pool.take(0, 9 * MB, &q, &m) == 0 && q == p && m == n && waits == 1);
        pool.give(0, q, m);
        assert(pool.take(0, 4 * MB, &q, &m) == 0 && q != p);                  // much smaller
        pool.give(0, q, m);
        assert(pool.take(0, 11 * MB, &q, &m) == 0 && q != p);                 // larger
        pool.give(0, q, m);
        assert(pool.drain(1) == 1 && pool.drain(0) == 3 && pool.drain(-1) == 0 && used == 0);
        // a wait that fails: the block stays, the caller gets one of its own
        assert(pool.take(0, MB, &p, &n) == 0);
        pool.give(0, p, n);
        wait_result = 9;
        assert(pool.take(0, MB, &q, &m) == 0 && q != p);
        wait_result = 0;
        Dev::free(q);
        assert(pool.take(0, MB, &q, &m) == 0 && q == p);
        Dev::free(q);
        assert(used == 0);
    }
    {   // at most kBlocks blocks and kBytes; a larger block evicts nothing
        Pool pool;
        std::vector<std::pair<void *, size_t>> v(12);
        for (auto &e : v) assert(pool.take(0, MB, &e.first, &e.second) == 0);
        for (auto &e : v) pool.give(0, e.first, e.second);
        assert(used == Pool::kBlocks * MB && live.count(v[11].first) && !live.count(v[0].first));
        assert(pool.take(0, Pool::kBytes + MB, &p, &n) == 0);
        pool.give(0, p, n);
        assert(used == Pool::kBlocks * MB);
        assert(pool.take(0, Pool::kBytes - 2 * MB, &p, &n) == 0);
        pool.give(0, p, n);
        assert(used <= Pool::kBytes);
        assert(pool.drain(-1) == 3 && used == 0);
    }
    {   // memory runs out: the idle blocks of the device go back, once
        Pool pool;
        capacity = 100 * MB;
        assert(pool.take(0, 60 * MB, &p, &n) == 0);
        pool.give(0, p, n);
        assert(pool.alloc(0, &q, 70 * MB) == 0 && used == 70 * MB);           // a workspace
        assert(pool.alloc(0, &p, 70 * MB) == Dev::no_memory && p == nullptr);
        Dev::free(q);
        assert(pool.take(0, 60 * MB, &p, &n) == 0);
        pool.give(0, p, n);
        assert(pool.take(0, 90 * MB, &q, &m) == 0 && used == 90 * MB);        // another plan
        pool.give(0, q, m);
        assert(pool.alloc(0, &p, 7) == 5 && p == nullptr && used == 90 * MB); // not out of memory
        assert(pool.drain(0) == 1 && used == 0);
        capacity = ~(size_t)0;
    }
    {   // threads
        Pool pool;
        std::vector<std::thread> t;
        for (int i = 0; i < 8; ++i)
            t.emplace_back([&pool, i] {
                for (int k = 0; k < 2000; ++k) {
                    void *p;
                    size_t n;
                    assert(pool.take(i & 1, (size_t)(1 + (k * 7 + i) % 5) * MB, &p, &n) == 0);
                    if (k % 50 == 0) pool.drain(i & 1);
                    pool.give(i & 1, p, n);
                }
            });
        for (auto &e : t) e.join();
        pool.drain(-1);
        assert(used == 0 && live.empty());
    }
    std::puts("pool ok");
}
"""


def test_block_pool(tmp_path):
    src, exe = tmp_path / "pool.cpp", tmp_path / "pool"
    src.write_text(PROGRAM)
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-pthread", "-fsanitize=address,undefined",
                        "-I", B.CSRC, str(src), "-o", str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120,
                       env={**os.environ, "LD_PRELOAD": ""})
    assert r.returncode == 0 and "pool ok" in r.stdout, r.stdout + r.stderr


def test_every_allocation_can_take_idle_blocks_back():
    """No allocation of the library goes past the pool's retry."""
    for name in sorted(os.listdir(B.CSRC)):
        text = open(os.path.join(B.CSRC, name)).read()
        if name == "abi.cpp":
            a, b = text.index("struct HipDev {"), text.index("BlockPool<HipDev> &block_pool()")
            text = text[:a] + text[b:]
        assert "hipMalloc(" not in text, name


def test_trim_without_plans():
    from paper_2503_18479_amd import trim
    trim()
    trim()
