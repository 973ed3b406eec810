"""The word that the K slabs of a tile meet at (csrc/any4_splitk.h), on the CPU: the function's own text, compiled for the host with
every access to the word a point where another slab may go on, and orders of those accesses tried, all of them for few slabs.  Whatever the order and
whatever the word held, waiting slabs included that look once or not at all: nobody adds before all have come, every part is added, and the
word is clean for the next meeting."""
import os
import re
import shutil
import subprocess

import pytest

HEADER = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2507_04610_amd", "csrc", "any4_splitk.h")

PROGRAM = r"""
#include <cstddef>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <ucontext.h>
#include <vector>
#define __device__
#define __host__
#define __forceinline__ inline
#define __HIP_MEMORY_SCOPE_AGENT 0
static void turn();                                       // the other slabs may go on here
template <class T, class V> T fetch_add(T* p, V v) { turn(); T o = *p; *p += v; return o; }
template <class T, class V> T fetch_or(T* p, V v) { turn(); T o = *p; *p |= v; return o; }
template <class T, class V> T fetch_and(T* p, V v) { turn(); T o = *p; *p &= v; return o; }
template <class T> T load(T* p) { turn(); return *p; }
template <class T, class V> void store(T* p, V v) { turn(); *p = (T)v; }
template <class T, class V> bool cas(T* p, T* e, V v) { turn(); if (*p == *e) { *p = (T)v; return true; } *e = *p; return false; }
#define __hip_atomic_fetch_add(p, v, o, s) fetch_add(p, v)
#define __hip_atomic_fetch_or(p, v, o, s) fetch_or(p, v)
#define __hip_atomic_fetch_and(p, v, o, s) fetch_and(p, v)
#define __hip_atomic_load(p, o, s) load(const_cast<std::remove_const_t<std::remove_pointer_t<decltype(p)>>*>(p))
#define __hip_atomic_store(p, v, o, s) store(p, v)
#define __hip_atomic_compare_exchange_strong(p, e, v, o, f, s) cas(p, e, v)
#define __builtin_amdgcn_s_sleep(n) ((void)0)
#include <type_traits>
//HEADER//
using namespace any4;

constexpr int kMax = 10;
static ucontext_t main_ctx, ctx[kMax];
static std::vector<char> stack_[kMax];
static int now, slabs_, parts_, looks_;
static bool begun[kMax], over[kMax], early;
static uint32_t got[kMax];
static unsigned long long word;

static void turn() { swapcontext(&ctx[now], &main_ctx); begun[now] = true; }
static void body(int k) {
    got[k] = meet(&word, slabs_, parts_, k, looks_);
    if (got[k]) for (int i = 0; i < slabs_; ++i) early |= !begun[i];       // (a slab's sums are out before its first access)
    over[k] = true;
    swapcontext(&ctx[k], &main_ctx);
}

// one run that follows `path` (which of the slabs still under way goes on) and then always the first; how many there were at each turn
static void run(unsigned long long start, const std::vector<int>& path, std::vector<int>& width) {
    word = start; early = false; width.clear();
    for (int k = 0; k < slabs_; ++k) {
        begun[k] = over[k] = false; got[k] = 0;
        getcontext(&ctx[k]);
        stack_[k].resize(64 << 10);
        ctx[k].uc_stack.ss_sp = stack_[k].data(); ctx[k].uc_stack.ss_size = stack_[k].size(); ctx[k].uc_link = &main_ctx;
        makecontext(&ctx[k], (void (*)())body, 1, k);
        now = k; swapcontext(&main_ctx, &ctx[k]);         // up to its first access
    }
    for (;;) {
        int live[kMax], n = 0;
        for (int k = 0; k < slabs_; ++k) if (!over[k]) live[n++] = k;
        if (!n) return;
        const size_t at = width.size();
        width.push_back(n);
        now = live[at < path.size() ? path[at] % n : 0];
        swapcontext(&main_ctx, &ctx[now]);
    }
}

int main(int argc, char** argv) {
    slabs_ = atoi(argv[1]); looks_ = atoi(argv[2]);
    const long most = atol(argv[3]);                      // orders; more: random ones
    parts_ = slabs_ < kMaxParts ? slabs_ : kMaxParts;
    constexpr unsigned long long T = kMeetTag, turn1 = 1ull << 16;
    const struct { unsigned long long w; bool once; } words[] = {
        {T, true}, {T | turn1, true}, {0, true}, {~0ull, true}, {0xA5A5A5A5A5A5A5A5ull, true}, {T - 1, true}, {0x00A4C0DE5EED1700ull, true},
        {T | 0xFF, false}, {T | 0xFFFF, true}, {T | turn1 | 0xFFFF, true}, {T | 0xFF00, false}, {T | 0x0300, false}, {T | turn1 | (unsigned)slabs_, true}};
    long total = 0;
    for (const auto& w : words) {
        std::vector<int> path, width;
        for (long n = 0; n < most; ++n, ++total) {
            run(w.w, path, width);
            int adders[8] = {0};
            for (int k = 0; k < slabs_; ++k) for (int p = 0; p < 8; ++p) adders[p] += got[k] >> p & 1;
            bool ok = !early && (word >> 17) == (T >> 17) && (word & 0xFFFF) == 0;
            for (int p = 0; p < parts_; ++p) ok &= w.once ? adders[p] == 1 : adders[p] >= 1;
            if (!ok) {
                printf("slabs %d looks %d start %016llx end %016llx early %d adders", slabs_, looks_, w.w, word, early);
                for (int p = 0; p < parts_; ++p) printf(" %d", adders[p]);
                printf("\n");
                return 1;
            }
            if (argc > 4) {                               // random orders
                path.assign(width.size() + 8, 0);
                for (size_t i = 0; i < path.size(); ++i) path[i] = i < width.size() ? rand() % width[i] : 0;
                continue;
            }
            path.resize(width.size(), 0);
            int i = (int)path.size() - 1;
            while (i >= 0 && path[i] + 1 >= width[i]) --i;
            if (i < 0) break;
            ++path[i];
            path.resize(i + 1);
        }
    }
    printf("%ld orders\n", total);
    return 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("no host compiler")
    text = re.sub(r"^#(include|pragma).*$", "", open(HEADER).read(), flags=re.M)
    d = tmp_path_factory.mktemp("meeting")
    src, exe = str(d / "meeting.cpp"), str(d / "meeting")
    open(src, "w").write(PROGRAM.replace("//HEADER//", text))
    subprocess.run(["g++", "-std=c++17", "-O1", "-w", src, "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("slabs,looks", ((2, 0), (2, 1), (2, 2), (3, 0)))
def test_every_order(program, slabs, looks):
    r = subprocess.run([program, str(slabs), str(looks), "1000000"], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr


@pytest.mark.parametrize("slabs,looks", ((3, 1), (4, 0), (5, 2), (8, 1), (9, 0), (10, 3)))
def test_random_orders(program, slabs, looks):
    """more slabs than can be tried in every order; as many as parts, and more"""
    r = subprocess.run([program, str(slabs), str(looks), "4000", "random"], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
