"""The dispatch rules of ad_internal.h that depend on sizes alone, compiled for
the host (no GPU needed)."""
import shutil
import subprocess

import pytest

from paper_1004_1932_amd import build

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include "ad_internal.h"
int main(int argc, char** argv) {
  for (int a = 1; a < argc; ++a) {
    long long v[4] = {0, 0, 0, 0};
    char name[64];
    std::sscanf(argv[a], "%63[^:]:%lld:%lld:%lld:%lld", name, v, v + 1, v + 2, v + 3);
    long long r = -1;
    if (!std::strcmp(name, "f64_by_threads")) r = ad::f64_by_threads((int)v[0], (int)v[1], (int)v[2]);
    if (!std::strcmp(name, "sym_takes")) r = ad::sym_takes((int)v[0], (int)v[1], (int)v[2]);
    std::printf("%lld\n", r);
  }
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    if not shutil.which(build.HIPCC):
        pytest.skip("needs hipcc")
    d = tmp_path_factory.mktemp("rules")
    (d / "rules.hip").write_text(PROGRAM)
    subprocess.run([build.HIPCC, "--offload-host-only", "-std=c++17", f"-I{build.CSRC}", str(d / "rules.hip"), "-o",
                    str(d / "rules")], check=True, capture_output=True)

    def call(name, *args):
        out = subprocess.run([str(d / "rules"), ":".join([name, *map(str, args)])], check=True, capture_output=True,
                             text=True)
        return int(out.stdout)
    return call


def test_fp64_ensembles_take_threads_only_where_no_system_outlasts_the_others(rule):
    def threads(sizes):
        return bool(rule("f64_by_threads", len(sizes), 2 * sum(sizes), 2 * max(sizes)))

    assert threads([1] * 4096) and threads([8] * 4096) and threads([32] * 4096) and threads([1] * 30000)
    assert threads([20, 40] * 2048) and threads([8] * 4095 + [16])
    assert not threads([1] * 4095) and not threads([33] * 4096)
    assert not threads([8] * 4095 + [2000]) and not threads([1] * 4095 + [2000])
    assert not threads([1] * 8191 + [200]) and not threads([20] * 4090 + [200] * 10)
    assert not threads([8] * 4095 + [60]) and not threads([1] * 4095 + [16])
