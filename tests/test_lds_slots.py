"""The LDS slots of the line transforms' exchanges (CPU-only: a host program
lists them).  LDS serves 8-byte reads 32 lanes, 8-byte writes 16 lanes and
4-byte accesses 32 lanes at a time; lanes served together must differ in the
slot's low 5, 4 and 5 bits.  Checked at every line length whose lines fill
whole groups of 32 lanes: every access but the writes of pass 0 outside the
split precisions, which take two turns, and no two points in one slot or
beyond the line's LDS."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2604_03585_amd", "csrc")
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"

pytestmark = pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")

PROGRAM = r"""
#include "mfma_fft.hpp"
#include <cstdio>
#include <set>
using namespace sar;

// most lanes of `group` served together that share a slot modulo `banks`
template <class F> int ways(int lanes, int group, int banks, F slot)
{
    int worst = 0;
    for (int g = 0; g < lanes; g += group) {
        int n[64] = {};
        for (int l = g; l < g + group; ++l) {
            const int k = ++n[slot(l) % banks];
            worst = k > worst ? k : worst;
        }
    }
    return worst;
}
template <int N, int P> void pass()
{
    using G = LineGeom<N>;
    if constexpr (P < G::NFULL && P < G::NP - 1) {
        constexpr int T = G::T, NS = G::span(P);
        int w8 = 0, r8 = 0, w4 = 0, r4 = 0;
        std::set<int> s8, s4;
        bool same = true;
        for (int i = 0; i < 16; ++i) {
            auto base = [](int t) { return (t / NS) * NS * 16 + (t & (NS - 1)); };
            auto m = [](int v, int w) { return v > w ? v : w; };
            w8 = m(w8, ways(T, 16, 16, [&](int t) { return lds_out<NS, P>(base(t), i); }));
            r8 = m(r8, ways(T, 32, 32, [&](int t) { return lds_in<T, P>(t, i); }));
            w4 = m(w4, ways(T, 32, 32, [&](int t) { return half_out<NS, P>(base(t), i); }));
            r4 = m(r4, ways(T, 32, 32, [&](int t) { return half_in<T, P>(t, i); }));
            for (int t = 0; t < T; ++t) {
                s8.insert(lds_in<T, P>(t, i));
                s4.insert(half_in<T, P>(t, i));
                same &= lds_in<T, P>(t, i) == lds_slot<P>(t + i * T) && half_in<T, P>(t, i) == half_slot<P>(t + i * T);
                same &= lds_out<NS, P>(base(t), i) == lds_slot<P>(base(t) + i * NS);
                same &= half_out<NS, P>(base(t), i) == half_slot<P>(base(t) + i * NS);
            }
        }
        std::printf("%d %d %d %d %d %d %d\n", N, P, w8, r8, w4, r4,
                    same && (int)s8.size() == N && (int)s4.size() == N && *s8.rbegin() < G::LDS && *s4.rbegin() < G::LDS);
        pass<N, P + 1>();
    }
}
template <int N> void mfma()
{
    using G = LineGeom<N>;
    int w = 0, r = 0;
    std::set<int> s;
    for (int e = 0; e < N; ++e) s.insert(mf_slot<N>(e));
    auto m = [](int v, int u) { return v > u ? v : u; };
    for (int j = 0; j < G::T; j += 16)
        for (int i = 0; i < 4; ++i) {
            r = m(r, ways(64, 32, 32, [&](int l) { return mf_slot<N>(j + (l & 15) + (4 * (l >> 4) + i) * G::T); }));
            for (int ns = 1; ns * 16 <= N; ns *= 16)
                w = m(w, ways(64, 16, 16, [&](int l) {
                    const int b = j + (l & 15);
                    return mf_slot<N>((b / ns) * ns * 16 + (b & (ns - 1)) + (4 * (l >> 4) + i) * ns);
                }));
        }
    std::printf("%d -1 %d %d 1 1 %d\n", N, w, r, (int)s.size() == N && *s.rbegin() < N);
}
int main()
{
    pass<512, 0>(); pass<1024, 0>(); pass<2048, 0>(); pass<4096, 0>(); pass<8192, 0>(); pass<16384, 0>();
    mfma<1024>(); mfma<2048>(); mfma<4096>(); mfma<8192>(); mfma<16384>();
}
"""


def test_slots_of_lanes_served_together(tmp_path):
    (tmp_path / "slots.hip").write_text(PROGRAM)
    r = subprocess.run([HIPCC, "-O1", "-std=c++17", "--offload-arch=gfx950", "-I", CSRC, str(tmp_path / "slots.hip"),
                        "-o", str(tmp_path / "slots")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    rows = [tuple(map(int, l.split())) for l in subprocess.run(
        [str(tmp_path / "slots")], capture_output=True, text=True, check=True).stdout.splitlines()]
    assert len(rows) == 14 + 5                      # exchanges of the six lengths, split lines of five
    for n, p, w8, r8, w4, r4, valid in rows:
        assert valid, (n, p)
        assert (r8, r4) == (1, 1) and w8 == w4 == (2 if p == 0 else 1), (n, p, w8, r8, w4, r4)
