"""The meeting of a cut row's parts (csrc/meet.hiph), compiled for the host and run in every order in which two and three
workgroups can come to their words of the slots, and in random orders for more: each part is a coroutine that hands over before
every access, which is what being switched out there amounts to.  Whatever a slot held before, exactly one part writes the row, with
all of it in the sum, and no sum is left behind."""
import os
import subprocess

import pytest

import paper_2403_17017_amd as S

DRIVER = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <ucontext.h>
#include <vector>
#define __device__
#define __forceinline__ inline
unsigned long wall_clock64();            // for a bound by time, should there be one: time flies while others run
#include "meet.hiph"

using seer::Meet;
typedef unsigned long long Word;

struct Part { ucontext_t ctx; std::vector<char> stack; bool over; uint32_t tile; float v; };
static std::vector<Part> parts;
static ucontext_t home;
static int running;
static Meet meet;
static uint32_t ts, te;
static float y;
static unsigned long model_clock;
static void hand_over() { model_clock += 1000000; swapcontext(&parts[running].ctx, &home); }
unsigned long wall_clock64() { hand_over(); return model_clock; }

struct Words {
    static Word exchange(Word *w, Word v) { hand_over(); const Word o = *w; *w = v; return o; }
    static Word look(Word *w) { hand_over(); return *w; }
};

static int writes;
static void body(int i)
{
    Part &p = parts[i];
    const float none = -1.f;
    float mine = none;
    seer::meet_end<Words>(meet, seer::meet_begin<Words>(meet, p.v, ts, te, p.tile), ts, te, &mine);
    if (mine != none) { ++writes; y = mine; }
    p.over = true;
}

// One run; `choose` picks among the parts that are not over.  The row's tiles are [ts, te].
template <class Choose> static bool run(std::vector<Word> &slots, Choose choose, bool rest = true)
{
    const int n = (int)(te - ts) + 1;
    meet.slots = slots.data();
    writes = 0;
    if ((int)parts.size() < n) parts.resize(n);
    float all = 0;
    for (int i = 0; i < n; ++i) {
        Part &p = parts[i];
        if (p.stack.empty()) p.stack.resize(65536);
        getcontext(&p.ctx);
        p.ctx.uc_stack.ss_sp = p.stack.data();
        p.ctx.uc_stack.ss_size = p.stack.size();
        p.ctx.uc_link = &home;
        p.over = false;
        p.tile = ts + (uint32_t)i;
        p.v = (float)(1 << i);                       // a part that is lost or doubled shows
        all += p.v;
        makecontext(&p.ctx, (void (*)())body, 1, i);
    }
    for (;;) {
        std::vector<int> can;
        for (int i = 0; i < n; ++i) if (!parts[i].over) can.push_back(i);
        if (can.empty()) break;
        running = can[choose((int)can.size())];
        swapcontext(&home, &parts[running].ctx);
    }
    bool ok = writes == 1 && y == all;
    for (size_t b = 0; rest && b < slots.size() / 8; ++b)           // only this row's boundaries
        if (b + 1 > ts && b + 1 <= te && slots[8 * b] != 0) ok = false;
    if (!ok) std::printf("row over tiles %u..%u: %d writes, sum %g of %g\n", ts, te, writes, y, all);
    return ok;
}

// every order: the choices of the run before, the last one that can be raised by one more
static long every(const std::vector<Word> &before, int &bad)
{
    std::vector<int> path, width;
    long runs = 0;
    for (;;) {
        size_t at = 0;
        std::vector<Word> slots = before;
        if (!run(slots, [&](int n) {
                if (at == path.size()) { path.push_back(0); width.push_back(n); }
                return path[at++];
            })) ++bad;
        ++runs;
        path.resize(at); width.resize(at);
        while (!path.empty() && path.back() + 1 == width.back()) { path.pop_back(); width.pop_back(); }
        if (path.empty()) return runs;
        ++path.back();
    }
}

static Word word(uint32_t mark, uint32_t low) { return (Word)mark << 32 | low; }

int main(int, char **argv)
{
    std::mt19937 rng(7);
    const std::vector<Word> at_rest(8 * 64);
    int bad = 0;
    meet.mark = 0xABCD1235u;
    meet.proof = 0x13579BDFu;
    const char *what = argv[1];
    if (!std::strcmp(what, "orders")) {
        long runs = 0;
        for (uint32_t from = 0; from < 8; ++from)
            for (uint32_t more = 1; more <= 2; ++more) {
                ts = from; te = from + more;
                runs += every(at_rest, bad);
            }
        std::printf("%ld orders\n", runs);
    } else if (!std::strcmp(what, "many")) {
        for (int k = 0; k < 20000; ++k) {
            ts = rng() % 20; te = ts + 1 + rng() % 12;
            std::vector<Word> slots = at_rest;
            if (!run(slots, [&](int n) { return (int)(rng() % n); })) ++bad;
        }
    } else if (!std::strcmp(what, "anything")) {
        for (int k = 0; k < 4000; ++k) {
            ts = rng() % 20; te = ts + 1 + rng() % 6;
            std::vector<Word> slots = at_rest;
            for (Word &w : slots) w = (Word)rng() << 32 | rng();
            if (k & 1)                                   // the mark, by chance, over something that is not a sum
                for (size_t b = 0; b < slots.size() / 8; ++b) slots[8 * b] = word(meet.mark, rng());
            // one part at a time for a while, so that some come to the end of their looks
            int left = 0, who = 0;
            if (!run(slots, [&](int n) {
                    if (left-- <= 0 || who >= n) { left = (int)(rng() % (k & 2 ? 600 : 3)); who = (int)(rng() % n); }
                    return who;
                })) ++bad;
            if (!run(slots, [&](int n) { return (int)(rng() % n); })) ++bad;       // and the next product
        }
    } else if (!std::strcmp(what, "left over")) {
        // sums of an earlier call in any slots, as two calls at a time leave them, then calls in order
        for (int k = 0; k < 4000; ++k) {
            ts = rng() % 20; te = ts + 1 + rng() % 6;
            std::vector<Word> slots = at_rest;
            const uint64_t random = (uint64_t)rng() << 32 | rng();
            const uint64_t call = k % 5 == 0 ? (0ull - random) / 3 : rng();
            const Meet old = seer::meet_of_call(slots.data(), random, call);
            for (size_t b = 0; b < slots.size() / 8; ++b)
                if (rng() % 2) {
                    const uint32_t bits = __builtin_bit_cast(uint32_t, 1e6f + (float)(rng() % 1000));
                    slots[8 * b] = word(old.mark, bits);
                    slots[8 * b + 1] = word(old.proof, bits);
                }
            for (uint64_t later = 1; later < 4; ++later) {
                meet = seer::meet_of_call(slots.data(), random, call + later);
                if (!run(slots, [&](int n) { return (int)(rng() % n); })) ++bad;
            }
            meet = old;                                  // a replay of the earlier call after them
            if (!run(slots, [&](int n) { return (int)(rng() % n); })) ++bad;
        }
    } else if (!std::strcmp(what, "marks")) {
        for (int k = 0; k < 200000; ++k) {
            const uint64_t random = (uint64_t)rng() << 32 | rng(), call = rng(), apart = 1 + rng() % 100000;
            const Meet a = seer::meet_of_call(nullptr, random, call), b = seer::meet_of_call(nullptr, random, call + apart);
            if ((a.mark == b.mark && a.proof == b.proof) || a.mark == 0 || b.mark == 0) ++bad;
        }
    } else {
        return 2;
    }
    return bad != 0;
}
"""


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    d = tmp_path_factory.mktemp("meetings")
    (d / "driver.cpp").write_text(DRIVER)
    csrc = os.path.join(os.path.dirname(os.path.abspath(S.__file__)), "csrc")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-x", "c++", "-I", csrc, "-o", str(d / "driver"), str(d / "driver.cpp")])
    return str(d / "driver")


@pytest.mark.parametrize("what", ["orders", "many", "anything", "left over", "marks"])
def test_cut_rows_meet_in_any_order(driver, what):
    out = subprocess.run([driver, what], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stdout[-2000:]
