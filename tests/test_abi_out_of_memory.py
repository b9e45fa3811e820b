"""C entry points report that host memory ran out; no C++ exception leaves
them (host code, no GPU)."""

import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

DRIVER = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <vector>
#include "sacx.h"

static bool refuse = false;
void *operator new(std::size_t n) {
    void *p = refuse && n > 65536 ? nullptr : std::malloc(n);
    if (!p) throw std::bad_alloc();
    return p;
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, std::size_t) noexcept { std::free(p); }

int main() {
    const int n = 20000;
    sacx_params p;
    std::memset(&p, 0, sizeof(p));
    p.gamma = 5.0 / 3.0; p.cfl = 0.3; p.hd_on = 1; p.hd_cross_on = 1;
    std::vector<sacx_grid> g(n, sacx_grid{16, 16, 0.0, 1.0, 0.0, 1.0, SACX_FP64, 0});
    std::vector<sacx_params> q(n, p);
    size_t bytes = 0, again = 0;
    if (sacx_batch_workspace_size(n, g.data(), q.data(), &bytes) != SACX_OK) return 1;
    refuse = true;
    const int rc = sacx_batch_workspace_size(n, g.data(), q.data(), &again);
    sacx_batch *b = nullptr;
    const int rc2 = sacx_batch_create(n, g.data(), q.data(), nullptr, (void *)(1 << 20), bytes, nullptr, &b);
    refuse = false;
    if (rc != SACX_EINVAL || !std::strstr(sacx_last_error(), "memory")) return 2;
    if (rc2 != SACX_EINVAL || b) return 3;
    if (sacx_batch_workspace_size(n, g.data(), q.data(), &again) != SACX_OK || again != bytes) return 4;
    std::printf("ok\n");
    return 0;
}
"""


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="no ROCm toolchain")
def test_out_of_host_memory_is_an_error_code(tmp_path):
    from paper_1710_06423_amd import build
    if not os.path.exists(build.LIB):
        build.build()
    src = tmp_path / "drv.cpp"
    src.write_text(DRIVER)
    exe = tmp_path / "drv"
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-I", build.INCLUDE, "-o", str(exe), str(src), build.LIB,
                        f"-Wl,-rpath,{os.path.dirname(build.LIB)}", "-Wl,--allow-shlib-undefined"],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip() == "ok", (r.returncode, r.stdout, r.stderr[-2000:])
