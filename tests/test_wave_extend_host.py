"""The wave's run extension (wave_extend in gwfa_kernels.hip) on the host: all
64 lanes take part in every exchange between lanes (an exchange under a branch
of some lanes reads nothing from the others), no lane reads a word outside the
packed stores, and every run gets its length.

The function's text is compiled for the host with the wave's lanes as
coroutines; each exchange is a switch point and checks that every lane stands
at the same one, and the window load checks its words against the store,
(N + 31) / 32 + 2 words for N bases.  Callers hand every lane's position
already advanced by one or two words, so a lane without a run may stand past
the store's end.  Lengths and counted words are compared with a plain loop."""
import re
import subprocess

import pytest

from paper_2206_13574_amd import build

_SRC = [s for s in build.sources() if s.endswith("gwfa_kernels.hip")][0]

_SHIM = r"""
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <algorithm>
#include <random>
#include <vector>
#include <ucontext.h>
using std::min; using std::max;
typedef unsigned long long ull;
#define __device__
#define __forceinline__ inline
#define __restrict__
struct Q { const ull* rd; };
static int cur, gen[64], site[2][64];
static ull slot[2][64];
static ucontext_t ctx[64], home;
static bool done[64];
static void next_lane() { const int me = cur; swapcontext(&ctx[me], &home); }
// every lane leaves its value, then all go on
static const ull* exchange(int line, ull x) {
    const int me = cur, b = gen[me]++ & 1;
    slot[b][me] = x;
    site[b][me] = line;
    next_lane();
    for (int i = 0; i < 64; ++i)
        if (site[b][i] != line || gen[i] < gen[me]) {
            printf("lanes %d and %d part at an exchange, line %d\n", me, i, line);
            exit(1);
        }
    return slot[b];
}
static int __lane_id() { return cur; }
static int __clzll(long long x) { return __builtin_clzll((ull)x); }
static ull ballot_at(int line, bool p) {
    const ull* s = exchange(line, p);
    ull m = 0;
    for (int i = 0; i < 64; ++i) m |= (s[i] & 1) << i;
    return m;
}
template <class T> static T lane_value(int line, T x, int l) { return (T)exchange(line, (ull)(int64_t)x)[l & 63]; }
#define __ballot(p) ballot_at(__LINE__, (p))
#define __shfl(x, l, w) lane_value(__LINE__, (x), (l))
#define __builtin_amdgcn_readlane(x, l) lane_value(__LINE__, (x), (l))
#define readlane64(x, l) lane_value(__LINE__, (int64_t)(x), (l))
static const ull* store[2];
static int64_t words[2];
static ull win32(const ull* w, int64_t p) {
    const int k = w == store[0] ? 0 : 1;
    const int64_t wi = p >> 5;
    if (p < 0 || wi + 1 >= words[k]) {
        printf("lane %d reads words %lld, %lld of %s store of %lld words\n", cur, (long long)wi, (long long)wi + 1,
               k ? "the label" : "the query", (long long)words[k]);
        exit(1);
    }
    const int sh = (int)(p & 31) * 2;
    return (w[wi] << sh) | ((w[wi + 1] >> 1) >> (63 - sh));
}
"""

_MAIN = r"""
static struct Lane { bool more; int64_t qp, sp; int32_t rem, ext; uint32_t chunks; } L[64];
static std::vector<ull> pack(const std::vector<int>& b) {
    std::vector<ull> w((b.size() + 31) / 32 + 2, 0);
    for (size_t i = 0; i < b.size(); ++i) w[i / 32] |= (ull)b[i] << (62 - 2 * (i % 32));
    return w;
}
static void lane_main() {
    Lane& l = L[cur];
    l.ext = wave_extend(store[1], Q{store[0]}, l.more, l.qp, l.sp, l.rem, l.chunks);
    done[cur] = true;
    next_lane();
}
int main() {
    std::mt19937 rng(17);
    static char stack[64][1 << 16];
    for (int round = 0; round < 960; ++round) {
        // one store's end is the other's, so that equal positions hold equal bases
        const int tail[3] = {0, 1, 31};
        const int n = 32 * (int)(4 + rng() % 60) + tail[round % 3];
        std::vector<int> q(n), s;
        for (auto& x : q) x = rng() & 3;
        s = q;
        const int errs = rng() % 4;
        for (int i = 0; i < errs; ++i) s[rng() % n] ^= 1;
        const std::vector<ull> qw = pack(q), sw = pack(s);
        store[0] = qw.data(); store[1] = sw.data();
        words[0] = qw.size(); words[1] = sw.size();
            const int step = round & 1 ? 32 : 64, runs = (round / 2) % 8;
        for (int l = 0; l < 64; ++l) {   // no run: anywhere a batch's lane may stand, the store's end among them
            const int at = rng() % 3 == 0 ? n - (int)(rng() % 3) : (int)(rng() % n);
            L[l] = Lane{false, at + step, at + step, at - n, 0, 0};
        }
        for (int i = 0; i < runs; ++i) {
            const int l = rng() % 64, at = rng() % (n - step);
            L[l] = Lane{true, at + step, at + step, 1 + (int)(rng() % (n - at - step)), 0, 0};
        }
        for (int l = 0; l < 64; ++l) {
            done[l] = false;
            gen[l] = 0;
            getcontext(&ctx[l]);
            ctx[l].uc_stack.ss_sp = stack[l];
            ctx[l].uc_stack.ss_size = sizeof stack[l];
            ctx[l].uc_link = &home;
            makecontext(&ctx[l], lane_main, 0);
        }
        for (bool any = true; any;) {
            any = false;
            for (cur = 0; cur < 64; ++cur)
                if (!done[cur]) { swapcontext(&home, &ctx[cur]); any = true; }
        }
        for (int l = 0; l < 64; ++l) {
            int e = 0;
            if (L[l].more)
                while (e < L[l].rem && q[L[l].qp + e] == s[L[l].sp + e]) ++e;
            const uint32_t w = !L[l].more ? 0 : e == L[l].rem ? (e + 31) / 32 : e / 32 + 1;
            if (e != L[l].ext || w != L[l].chunks) {
                printf("round %d lane %d: length %d (%d), words %u (%u)\n", round, l, L[l].ext, e, L[l].chunks, w);
                return 1;
            }
        }
    }
    printf("ok\n");
}
"""


def _function(text, name):
    """The definition of one device function."""
    a = re.search(r"^__device__[^;{]*\b" + name + r"\(", text, re.M).start()
    depth, i = 0, text.index("{", a)
    while True:
        depth += {"{": 1, "}": -1}.get(text[i], 0)
        i += 1
        if depth == 0:
            return text[a:i] + "\n"


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    d = tmp_path_factory.mktemp("wave_extend")
    (d / "t.cpp").write_text(_SHIM + _function(open(_SRC).read(), "wave_extend") + _MAIN)
    r = subprocess.run(["g++", "-O1", "-std=c++17", "-w", "-o", str(d / "t"), str(d / "t.cpp")], capture_output=True,
                       text=True)
    assert r.returncode == 0, r.stderr
    return subprocess.run([str(d / "t")], capture_output=True, text=True, timeout=120)


def test_runs_stay_in_the_stores_and_have_their_lengths(run):
    assert run.returncode == 0 and run.stdout == "ok\n", run.stdout + run.stderr
