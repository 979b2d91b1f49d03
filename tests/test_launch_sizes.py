"""Launches over the elements of a large model: HIP supports fewer than 2^32
threads along a grid dimension, and the split planes of 3 million rows of 1000
labels are 4.6e9 dwords, so fills and packing walk a capped grid."""

import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1806_06144_amd", "csrc")

PROGRAM = r"""
#include "launch.h"
#include <cstdio>
#include <cstdlib>
int main(int, char** argv) {
    std::printf("%u\n", ep::stride_grid(std::atoll(argv[1]), std::atoi(argv[2])));
}
"""


@pytest.fixture(scope="module")
def stride_grid(tmp_path_factory):
    d = tmp_path_factory.mktemp("launch")
    src, exe = d / "g.cpp", d / "g"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    return lambda blocks, threads: int(subprocess.run(
        [str(exe), str(blocks), str(threads)], check=True, capture_output=True, text=True).stdout)


@pytest.mark.parametrize("threads", [256, 1024])
@pytest.mark.parametrize("blocks", [0, 1, 1023, 1 << 20, (1 << 24) - 1, 1 << 24, 1 << 33])
def test_grids_stay_below_the_limit(stride_grid, blocks, threads):
    g = stride_grid(blocks, threads)
    assert g * threads < 1 << 32
    assert g == min(blocks, ((1 << 32) - 1) // threads)   # whole launches stay whole


def test_planes_of_three_million_rows(stride_grid):
    n, l = 3000000, 1000
    dwords = -(-n // 256) * 256 // 32 * -(-l // 16) * 3 * 1024 // 4
    assert -(-dwords // 256) * 256 >= 1 << 32             # (one thread a dword is refused)
    assert stride_grid(-(-dwords // 256), 256) * 256 < 1 << 32


@pytest.mark.parametrize("name,file", [("fill_kernel", "kernels.hip"),
                                       ("pack_weights_kernel", "skmv.hip"),
                                       ("pack_rows_kernel<true>", "skmv.hip"),
                                       ("pack_rows_kernel<false>", "skmv.hip")])
def test_their_launches_are_capped_and_walk(name, file):
    text = open(os.path.join(CSRC, file)).read()
    at = text.index(f"hipLaunchKernelGGL({name},")
    grid = text[at - 200:text.index(";", at)]
    assert "stride_grid(" in grid
    body = text[text.index(f" {name.split('<')[0]}("):]
    assert "+= " in body[:900] and "gridDim.x" in body[:900]


SPLITS = r"""
#include "launch.h"
#include <cmath>
#include <cstdio>
#include <vector>
typedef std::vector<std::pair<int64_t, int64_t>> List;
int main() {
    for (int64_t items = 1; items < 70000; items += items < 700 ? 1 : 997)
        for (int64_t most : {int64_t(1), int64_t(7), int64_t(512), int64_t(1) << 20}) {
            List a, b;
            ep::each_split(items, most, [&](int64_t p, int64_t per) { a.push_back({p, per}); });
            for (int64_t p = 1; p <= items && p <= most; ++p) {
                const int64_t per = (items + p - 1) / p;
                if ((items + per - 1) / per == p) b.push_back({p, per});
            }
            if (a != b || (double)a.size() > 2 * std::sqrt((double)items) + 1) {
                std::printf("items %lld most %lld: %zu and %zu\n", (long long)items,
                            (long long)most, a.size(), b.size());
                return 1;
            }
        }
}
"""


def test_split_counts_are_those_of_a_full_scan(tmp_path):
    src, exe = tmp_path / "s.cpp", tmp_path / "s"
    src.write_text(SPLITS)
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
    text = open(os.path.join(CSRC, "skmv.hip")).read()
    assert text.count("each_split(") == 2 and "++P" not in text


@pytest.mark.gpu
@pytest.mark.timeout(300)
def test_model_of_more_plane_dwords_than_threads():
    """Setup (zero planes), set_alpha (packed planes) and prediction of such a
    model; every plane past 2^32 dwords is in the last rows' weights."""
    import numpy as np
    import torch
    import paper_1806_06144_amd as ep
    n, d, l, nz, bw = 3000000, 8, 1000, 40, 2.0
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(5)
    X = torch.randn((n, d), device=dev, generator=gen)
    Z = torch.randn((nz, d), device=dev, generator=gen)
    ctx, _ = ep.ep_setup(X, n, d, l, "gaussian", bw, 64, 2, sub_idx=np.arange(64))
    try:
        out = torch.empty((nz, l), device=dev)
        ep.ep_predict(ctx, Z, nz, out)
        ep.ep_sync(ctx)
        assert float(out.abs().max()) == 0.0
        a = torch.zeros((n, l), device=dev)
        a[-300000:].normal_(generator=gen)
        ep.ep_set_alpha(ctx, a)
        ep.ep_predict(ctx, Z, nz, out)
        ep.ep_sync(ctx)
    finally:
        ep.ep_destroy(ctx)
    ref = torch.zeros((nz, l), dtype=torch.float64, device=dev)
    scale = torch.zeros((nz, l), dtype=torch.float64, device=dev)
    for c in range(n - 300000, n, 50000):
        d2 = torch.cdist(Z.double(), X[c:c + 50000].double()) ** 2
        K = torch.exp(-d2 / (2 * bw * bw))
        A = a[c:c + 50000].double()
        ref += K @ A
        scale += K @ A.abs()
    # a term's kernel value is off by a few roundings of its distance (8
    # features: 4 eps (|x|^2 + |z|^2) / (2 bw^2), below 30 eps here), a sum of
    # 3e5 terms in chains of at most 1e4 groups by less than that again
    assert float(((out - ref).abs() / scale).max()) < 60 * 2.0 ** -24
