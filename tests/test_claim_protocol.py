"""Host-side check of the device-driven solve's claim protocol (`pmf_claim.h`):
a model of its workgroups (look at the claim word, add to it, take, count the
finished entries and claim again, publish the next superstep), every atomic a
step of its own, is stepped through all interleavings of two or three
consecutive supersteps with different batches.  Every entry of every superstep
has to be taken exactly once, and no interleaving may come to a stop before
the end.  With workgroups that may give up whenever they look for work, a run
either is completed all the same or was never begun: no superstep is left
half done.  The header is compiled with the host compiler."""

import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1509_06004_amd", "csrc")

HARNESS = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <set>
#include <string>
#include <vector>
#include "pmf_claim.h"
using namespace pmf;
constexpr int kW = 3, kS = 3, kE = 9;  // workgroups, supersteps, entries at most
struct Step { int count, batch; };
// what a workgroup does next
enum Pc : uint8_t { kLook, kAdd, kClear, kRun, kBoth, kDoneOnly, kClaimOnly, kDecide, kZero, kMark, kPublish, kGone };
struct Group {
    Pc pc;
    uint8_t step, first, n, last;  // its task
    uint8_t added;                 // amount of the add under way
    uint8_t done;                  // reply of the done word
    uint64_t old;                  // reply of the claim word
    uint32_t hi;
};
struct State {
    uint64_t claim;
    uint8_t done, bit, over;
    uint8_t taken[kS][kE];
    Group g[kW];
};
std::vector<Step> steps;
const char *fail = nullptr;
bool give_up = false;  // a workgroup may leave whenever it looks for work

uint64_t word(int s, int own) { return (uint64_t)claim_hi(steps[s].count, s, steps[s].batch) << 32 | (unsigned)own; }
int step_of(uint32_t hi) { return (int)(hi >> kClCountBits) & (kClTags - 1); }

void take(Group &g, uint64_t old, int added) {
    const Claim c = claim_take(old, added);
    if (c.n == 0) { g.pc = kLook; g.n = 0; return; }
    g.hi = c.hi;
    g.step = (uint8_t)step_of(c.hi);
    g.first = (uint8_t)c.first;
    g.n = (uint8_t)c.n;
    g.last = c.last;
    g.pc = c.last ? kClear : kRun;
}

void run(State &st, Group &g) {
    if (g.first + g.n > steps[g.step].count) fail = "past the end";
    for (int i = 0; i < g.n && !fail; ++i)
        if (++st.taken[g.step][g.first + i] > 1) fail = "an entry taken twice";
}

// The successors of workgroup i: the same state with its next step done.
void advance(const State &s0, int i, std::vector<State> &out) {
    State s = s0;
    Group &g = s.g[i];
    switch (g.pc) {
        case kLook:
            if (s.over) { g = Group{}; g.pc = kGone; break; }
            if (give_up) {
                State t = s;
                t.g[i] = Group{};
                t.g[i].pc = kGone;
                out.push_back(t);
            }
            if (!s.bit) return;  // polls
            g.hi = (uint32_t)(s.claim >> 32);
            if ((int)(uint32_t)s.claim >= claim_count(g.hi)) return;  // nothing left: polls
            g.added = (uint8_t)claim_batch(g.hi);
            g.pc = kAdd;
            break;
        case kAdd: {
            const uint64_t old = s.claim;
            s.claim += g.added;
            const int added = g.added;
            g = Group{};
            take(g, old, added);
            break;
        }
        case kClear: s.bit = 0; g.pc = kRun; break;
        case kRun: run(s, g); g.added = (uint8_t)claim_batch(g.hi); g.pc = kBoth; break;
        case kBoth: {  // the two adds of one instruction arrive in either order
            State t = s;
            Group &f = t.g[i];
            f.done = t.done; t.done = (uint8_t)(t.done + f.n); f.pc = kClaimOnly;
            out.push_back(t);
            g.old = s.claim; s.claim += g.added; g.pc = kDoneOnly;
            break;
        }
        case kDoneOnly: g.done = s.done; s.done = (uint8_t)(s.done + g.n); g.pc = kDecide; break;
        case kClaimOnly: g.old = s.claim; s.claim += g.added; g.pc = kDecide; break;
        case kDecide: {
            const int d = g.done + g.n;
            if (d > claim_count(g.hi)) fail = "more done than listed";
            if (d == claim_count(g.hi)) {
                for (int e = 0; e < steps[g.step].count; ++e)
                    if (s.taken[g.step][e] != 1) fail = "completed with an entry not taken";
                if (g.step + 1 == (int)steps.size()) { s.over = 1; g = Group{}; g.pc = kGone; }
                else { const uint8_t n = (uint8_t)(g.step + 1); g = Group{}; g.step = n; g.pc = kZero; }
            } else {
                const uint64_t old = g.old;
                const int added = g.added;
                g = Group{};
                take(g, old, added);
            }
            break;
        }
        case kZero: s.done = 0; g.pc = kMark; break;
        case kMark: {
            const Step &p = steps[g.step];
            if (p.count > p.batch) s.bit = 1;
            g.pc = kPublish;
            break;
        }
        case kPublish: {
            const Step &p = steps[g.step];
            const int own = p.batch < p.count ? p.batch : p.count;
            s.claim = word(g.step, own);
            g.hi = (uint32_t)(s.claim >> 32);
            g.first = 0; g.n = (uint8_t)own; g.last = 0;
            g.pc = kRun;
            break;
        }
        case kGone: return;
    }
    out.push_back(s);
}

int main(int argc, char **argv) {
    const int nw = atoi(argv[1]);
    give_up = atoi(argv[2]) != 0;
    for (int a = 3; a + 1 < argc; a += 2) steps.push_back(Step{atoi(argv[a]), atoi(argv[a + 1])});
    State s0;
    std::memset(&s0, 0, sizeof(s0));
    s0.claim = word(0, 0);
    s0.bit = 1;
    for (int i = nw; i < kW; ++i) s0.g[i].pc = kGone;
    std::set<std::string> seen;
    std::vector<State> todo = {s0};
    seen.insert(std::string((const char *)&s0, sizeof(s0)));
    size_t ends = 0;
    std::vector<State> next;
    while (!todo.empty()) {
        const State s = todo.back();
        todo.pop_back();
        next.clear();
        for (int i = 0; i < kW; ++i) advance(s, i, next);
        if (fail) { printf("%s\n", fail); return 1; }
        if (next.empty()) {
            for (int i = 0; i < kW; ++i) if (s.g[i].pc != kGone) { printf("stopped before the end\n"); return 2; }
            size_t taken = 0, all = 0;
            for (size_t t = 0; t < steps.size(); ++t)
                for (int e = 0; e < steps[t].count; ++e) { ++all; taken += s.taken[t][e] == 1; }
            if (taken != all && !(give_up && taken == 0 && (uint32_t)s.claim == 0)) { printf("half done\n"); return 3; }
            ++ends;
        }
        for (State &n : next) {
            State c;  // no padding bytes of a copy in the key
            std::memset(&c, 0, sizeof(c));
            c.claim = n.claim; c.done = n.done; c.bit = n.bit; c.over = n.over;
            std::memcpy(c.taken, n.taken, sizeof(c.taken));
            for (int i = 0; i < kW; ++i) {
                Group &x = c.g[i], &y = n.g[i];
                x.pc = y.pc; x.step = y.step; x.first = y.first; x.n = y.n; x.last = y.last;
                x.added = y.added; x.done = y.done; x.old = y.old; x.hi = y.hi;
            }
            if (seen.insert(std::string((const char *)&c, sizeof(c))).second) todo.push_back(c);
        }
    }
    printf("%zu states, %zu ends\n", seen.size(), ends);
    return ends ? 0 : 4;
}
"""


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("needs a host C++ compiler")
    d = tmp_path_factory.mktemp("claim")
    src, exe = d / "claim_model.cpp", d / "claim_model"
    src.write_text(HARNESS)
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    return str(exe)


# (entries, batch) of consecutive supersteps: the batch grows, shrinks, divides
# the list and does not
RUNS = [[(4, 1), (4, 2)], [(4, 2), (9, 4)], [(5, 4), (6, 2)], [(5, 4), (3, 1)], [(2, 1), (6, 4)], [(6, 4), (5, 1)],
        [(3, 2), (3, 1), (3, 2)], [(4, 2), (1, 1), (7, 4)]]


@pytest.mark.parametrize("groups,give_up", [(2, 0), (3, 0), (3, 1)])
@pytest.mark.parametrize("run", RUNS, ids=str)
def test_every_entry_is_taken_once(model, run, groups, give_up):
    args = [str(groups), str(give_up)] + [str(x) for s in run for x in s]
    r = subprocess.run([model] + args, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, (r.returncode, r.stdout, r.stderr)


FIELDS = r"""
#include <initializer_list>
#include "pmf_claim.h"
using namespace pmf;
int main() {
    // the three fields of the high word keep apart at the ends of their ranges
    const int counts[] = {1, 2, 639, 640, kClCountMax}, batches[] = {1, 2, 15, kClBatchMax};
    for (int c : counts)
        for (int b : batches)
            for (int t : {0, 1, kClTags - 1, kClTags, 65535}) {
                const uint32_t hi = claim_hi(c, t, b);
                if (claim_count(hi) != c || claim_batch(hi) != b || hi == 0) return 1;
                if (hi == claim_hi(c, t + 1, b)) return 2;
                for (int added : {1, 3, 16})
                    for (int next : {0, c - 1, c, c + 7}) {
                        const Claim k = claim_take((uint64_t)hi << 32 | (unsigned)next, added);
                        const int left = c - next > 0 ? c - next : 0, n = added < left ? added : left;
                        if (k.n != n || k.hi != hi || (n && k.first != next) || k.last != (n && n == left)) return 3;
                    }
            }
    return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs a host C++ compiler")
def test_claim_word_fields(tmp_path):
    src, exe = tmp_path / "fields.cpp", tmp_path / "fields"
    src.write_text(FIELDS)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    assert subprocess.run([str(exe)]).returncode == 0
