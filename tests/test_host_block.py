"""Host memory that a blocking call reads back into (host_block.hpp): pinned blocks go from call to call, at most as many as are kept; one that a
copy may still go to is not handed on; where pinned memory is refused there is ordinary memory, and none of it stays."""
import subprocess

from paper_2510_24273_amd import build

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <atomic>
#include <thread>
#include <vector>
#include "host_block.hpp"
static std::atomic<int> made{0}, freed{0};
static bool refuse = false;
struct Alloc {
    static void* pin(size_t n) { if (refuse) return nullptr; ++made; return std::malloc(n); }
    static void unpin(void* p) { ++freed; std::free(p); }
};
typedef sals::HostBlock<Alloc, 4096, 2> Block;
#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)
int main()
{
    void* first;
    { Block b; first = b.p; CHECK(first && made == 1); std::memset(b.p, 1, 4096); b.idle = true; }
    CHECK(freed == 0);
    refuse = true;   // a kept one needs no new one
    { Block b; CHECK(b.p == first); Block c; CHECK(c.p && c.p != first && made == 1); std::memset(c.p, 2, 4096); b.idle = c.idle = true; }
    CHECK(freed == 0);
    refuse = false;
    { Block a, b, c; CHECK(made == 3); a.idle = b.idle = c.idle = true; }   // three at once, of which two are kept
    CHECK(freed == 1);
    { Block a, b; CHECK(made == 3); a.idle = true; }   // b: a copy may be under way
    CHECK(freed == 2);
    std::vector<std::thread> t;
    for (int k = 0; k < 4; ++k)
        t.emplace_back([] { for (int i = 0; i < 2000; ++i) { Block b; std::memset(b.p, i, 4096); b.idle = true; } });
    for (auto& x : t) x.join();
    CHECK(made - freed >= 1 && made - freed <= 2);
    std::printf("ok\n");
}
"""


def test_blocks(tmp_path):
    (tmp_path / "b.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-I", build.CSRC, "-o", str(tmp_path / "b"), str(tmp_path / "b.cpp")], check=True)
    assert subprocess.run([str(tmp_path / "b")], capture_output=True, text=True, timeout=60).stdout.strip() == "ok"
