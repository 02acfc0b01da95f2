"""Objects lent to threads (csrc/skim_lease.h), on the CPU: threads that come and go
share one, threads side by side get one each, and one that is dropped is not lent
again."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHECK = r"""
#include "skim_lease.h"
#include <atomic>
#include <cstdio>
#include <set>
#include <thread>
using namespace skim;
struct Box { std::atomic<int> users{0}; };
static std::atomic<int> made{0};
static LeasePool<Box> &pool = *new LeasePool<Box>;
static Box *box(bool drop = false) {
    thread_local Lease<Box> lease(pool);
    Box *b = lease.get([] { ++made; return new Box; });
    if (drop) lease.drop();
    return b;
}
int main() {
    for (int i = 0; i < 500; ++i) std::thread([] { box(); box(); }).join();
    if (made != 1) return std::printf("%d made for threads one after the other\n", (int)made), 1;
    std::atomic<int> shared{0}, there{0};
    std::thread t[8];
    for (auto &x : t)
        x = std::thread([&] {
            Box *b = box();
            if (b->users++) ++shared;
            ++there;
            while (there < 8) std::this_thread::yield();  // all hold one at once
            --b->users;
        });
    for (auto &x : t) x.join();
    if (shared || made > 8) return std::printf("%d shared, %d made\n", (int)shared, (int)made), 1;
    const int before = made;
    std::set<Box *> dropped;
    for (int i = 0; i < 8; ++i) std::thread([&] { dropped.insert(box(true)); }).join();
    Box *next = nullptr;
    std::thread([&] { next = box(); }).join();
    if (dropped.count(next) || made != before + 1) return std::puts("a dropped one was lent"), 1;
    std::puts("lent and given back");
    return 0;
}
"""


def test_threads_share_what_is_given_back(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ is not available")
    src, exe = tmp_path / "lease.cpp", tmp_path / "lease"
    src.write_text(CHECK)
    r = subprocess.run([gxx, "-O1", "-std=c++17", "-pthread", "-I" + os.path.join(ROOT, "paper_1408_6282_amd", "csrc"),
                        str(src), "-o", str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0, out.stdout
