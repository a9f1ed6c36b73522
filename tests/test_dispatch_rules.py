"""The lines that decide which form a call takes, asked on the CPU: the library's host side is compiled with a stand-in for its
kernels, so a rule can be checked on both sides of its line at any size."""
import os
import re
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    hipcc, rocm = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), os.environ.get("ROCM_PATH", "/opt/rocm")
    obj, exe = str(d / "rules.o"), str(d / "rules")
    subprocess.check_call([hipcc, "--offload-arch=gfx950", "--cuda-host-only", "-O0", "-std=c++17", "-x", "hip", "-c", "-o", obj,
                           os.path.join(HERE, "dispatch", "rules.cpp")], stderr=subprocess.DEVNULL)
    # the kernels' image, which nothing asks for
    name = re.search(r" U (__hip_fatbin\S*)", subprocess.check_output(["nm", obj], text=True)).group(1)
    (d / "image.c").write_text(f"const char {name}[4096] __attribute__((aligned(4096))) = {{0}};\n")
    subprocess.check_call(["g++", "-no-pie", "-o", exe, obj, "-x", "c", str(d / "image.c"), "-x", "none", f"-L{rocm}/lib", "-lamdhip64",
                           f"-Wl,-rpath,{rocm}/lib"])

    def f(what, K, n, storage="f32", *more):
        out = subprocess.check_output([exe, what, str(K), str(n), storage, *map(str, more)], text=True)
        return [int(a) for a in out.split()]
    return f


@pytest.mark.parametrize("K,n,main", [(3, 1 << 20, 1), (3, (1 << 20) + 1, 0), (7, 1 << 19, 1), (7, (1 << 19) + 1, 0), (15, 1 << 18, 1),
                                      (15, (1 << 18) + 1, 0), (31, 1 << 17, 1), (63, 1 << 16, 1), (63, (1 << 16) + 1, 0),
                                      (8, 465_920, 1), (8, 465_921, 0), (1, 1 << 21, 1), (64, 1000, 1)])
def test_a_mean_of_exactly_16_mib_stays_on_the_main_stream(ask, K, n, main):
    """(K + 1) n 4 bytes: lengths that meet the line exactly are those whose arenas get a row more."""
    on_main, split = ask("mean_on_main", K, n)
    assert on_main == main
    assert split == (4 if K >= 12 else 2 if K >= 8 and not main else 1)
