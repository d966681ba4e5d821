"""Where the initial condition's parts lie (a host build of the planner): inside what was lent or one block,
256-byte aligned, apart from each other while both are in use, and apart from what the call writes meanwhile."""
import os
import shutil
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

MAIN = r'''
#include <cstdio>
#include <cstdlib>
#include <vector>
using namespace cpic;
static size_t taken;
hipError_t cpic::pool_take(int, size_t bytes, PoolBlock* out) { taken = bytes; out->p = (void*)((size_t)9 << 40); out->bytes = bytes; return hipSuccess; }
void cpic::pool_give(int, PoolBlock) {}
#define FAIL(...) do { std::printf(__VA_ARGS__); std::exit(1); } while (0)
int main()
{
    long plans = 0;
    for (int N = 4; N <= 1024; N++) {
        int m = N;
        while (m % 2 == 0) m /= 2;
        while (m % 3 == 0) m /= 3;
        if (m != 1) continue;
        for (int nc = 2; nc <= 3; nc++) for (int f32 = 0; f32 < 2; f32++) for (int third = 0; third < 2; third++)
            for (int sheets : {1, 2, 7, 50, 400}) for (double uv : {0.0, 0.3, 2.0}) {
                const size_t V = (size_t)N * N, tsz = f32 ? 4 : 8, fb = (nc == 2 ? 20 : 68) * V * tsz;
                const size_t links = (nc == 2 ? 8 : 36) * V * tsz, mw = 8 * (nc == 2 ? 4 : 18) * V;
                char* const set[3] = {(char*)((size_t)1 << 40), (char*)((size_t)2 << 40), third ? (char*)((size_t)3 << 40) : nullptr};
                ICArgs a{};
                a.N = N; a.n_sheets = sheets; a.uvhat = uv;
                ICScratch mem(0);
                const size_t lk = f32 ? links : 0, rest = std::min(fb, (lk + 255) / 256 * 256);
                mem.lend(set[2], fb, ICScratch::kAll);
                mem.lend(set[1], fb, ICScratch::kAll);
                mem.lend(set[0], lk, ICScratch::only(ICScratch::kThroughout) | ICScratch::only(ICScratch::kBefore));
                mem.lend(set[0] + rest, fb - rest, ICScratch::only(ICScratch::kBefore));
                ICWork w{};
                taken = 0;
                if (ic_reserve(a, nc, f32, mem, &w) != hipSuccess) FAIL("%d %d refused\n", N, nc);
                plans++;
                // what the planner placed, and the phases (1 before, 2 after, 3 rounding) it is in use
                struct P { char* at; size_t n; unsigned when; };
                std::vector<P> ps;
                for (int k = 0; k < mem.nparts; k++) {
                    const auto s = mem.parts[k].span;
                    // (the Wilson lines are last read by pi(0), the double links by the rounding)
                    ps.push_back({mem.parts[k].at, mem.parts[k].bytes, s == ICScratch::kBefore ? 1u : s == ICScratch::kAfter ? 6u : 3u});
                }
                const size_t own = ps.size();
                // what the call itself writes: the fields (phi, E, pi) from the links on, and the links: solved in place, or rounded
                ps.push_back({set[0] + links, fb - links, 6u});
                ps.push_back({set[0], links, f32 ? 4u : 6u});
                for (size_t i = 0; i < ps.size(); i++) {
                    const P& p = ps[i];
                    if (i < own) {
                        if (!p.at || (size_t)p.at % 256) FAIL("%d nc %d f32 %d: part %zu unaligned or missing\n", N, nc, f32, i);
                        bool in = false;
                        for (char* s : set) in = in || (s && p.at >= s && p.at + p.n <= s + fb);
                        in = in || (p.at >= (char*)((size_t)9 << 40) && p.at + p.n <= (char*)((size_t)9 << 40) + taken);
                        if (!in) FAIL("%d nc %d f32 %d: part %zu out of range\n", N, nc, f32, i);
                    }
                    for (size_t j = 0; j < i; j++)
                        if ((p.when & ps[j].when) && p.at < ps[j].at + ps[j].n && ps[j].at < p.at + p.n)
                            FAIL("%d nc %d f32 %d third %d sheets %d: parts %zu and %zu overlap\n", N, nc, f32, third, sheets, i, j);
                }
                if (taken > std::max(kPoolBytes + 65536 * 16, f32 ? 2 * mw + 512 : 0) + mw) FAIL("%d: %zu bytes\n", N, taken);
            }
    }
    std::printf("%ld plans\n", plans);
}
'''


def test_parts_lie_apart(tmp_path):
    csrc = os.path.join(ROOT, "paper_2303_05599_amd", "csrc")
    (tmp_path / "main.hip").write_text('#include "%s"\n' % os.path.join(csrc, "ic.hip") + MAIN)
    exe = str(tmp_path / "plan")
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    r = subprocess.run([hipcc, "--offload-arch=gfx950", "-O1", "-std=c++17", "-w", "-I", csrc, "-o", exe, str(tmp_path / "main.hip")],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and "plans" in r.stdout, r.stdout + r.stderr
