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


def test_symmetric_pair_sum_within_its_sizes(rule):
    for N in (8704, 65536, 585000):
        assert rule("sym_takes", N, 1, 0) and rule("sym_takes", N, 0, 1)
    for N in (8702, 585002, 1 << 20, 1 << 23):
        assert not rule("sym_takes", N, 1, 0) and not rule("sym_takes", N, 0, 1) and not rule("sym_takes", N, 0, 0)


def test_workspace_of_the_largest_systems_grows_linearly():
    """One FP32C system, default launch: what an ordered pair sum needs. Its
    partial sums per lower block would be 13 GB at 2^20 spheres."""
    from paper_1004_1932_amd import binding as B
    from workload import Params

    def size(N):
        ctx = B.ad_create(B.make_params(Params(), "fp32c"), [N // 2])
        n = B.ad_workspace_size(ctx)
        B.ad_destroy(ctx)
        return n

    assert size(1 << 20) <= 1000 * (1 << 20)
    assert size(1 << 21) <= 2.1 * size(1 << 20)
    assert size(1 << 19) <= 5 << 30


def test_autotuner_knows_which_steps_the_symmetric_pair_sum_takes(rule):
    from dataclasses import replace

    from paper_1004_1932_amd import autotune as A
    from paper_1004_1932_amd import binding as B
    from workload import Params
    for N in (8702, 8704, 13310, 13312, 60000, 585000, 585002):
        for posmode in (B.AD_POS_HILO, B.AD_POS_SINGLE):
            for ks in (0.0, 1.0):
                want = rule("sym_takes", N, int(posmode == B.AD_POS_HILO), int(ks != 0.0))
                assert A.step_ignores_shape(replace(Params(), steric_k=ks), [N // 2], dict(posmode=posmode)) == want
