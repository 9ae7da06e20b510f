"""What bench.py says of the matrix-product kernels is about the kernels that run."""

import os
import re
import shutil

import bench
from paper_2403_11204_amd import api

CSRC = os.path.join(bench.ROOT, "paper_2403_11204_amd", "csrc")


def test_named_kernels_exist_and_take_most_of_the_products():
    defined = set()
    for name in os.listdir(CSRC):
        defined |= set(re.findall(r"__global__[^;{]*?\b(\w+_kernel)\(", open(os.path.join(CSRC, name)).read()))
    for config, cfg in bench.CONFIGS.items():
        named = bench.PRODUCT_KERNELS[config].split(", ")
        assert set(named) <= defined, config
        work = {"long": 0, "big": 0, "other": 0}
        B = cfg["batch"]
        for widths, *_ in cfg["segs"]:
            for l, (k, n) in enumerate(zip(widths, widths[1:])):
                for M, N, K in [(B, n, k), (n, k, B)] + ([(B, k, n)] if l else []):
                    big = cfg["dtype"] == api.BF16 and -(-M // 256) * -(-N // 256) >= 224
                    work["long" if big and K >= 3072 else "big" if big else "other"] += M * N * K
        most = max(work, key=work.get)
        assert (named[0] == "gemm_nt_long_kernel") == (most == "long"), (config, work)


def test_traffic_is_given_for_the_measured_sources_only(tmp_path, monkeypatch):
    assert bench.gemm_traffic(0) is None
    csrc = tmp_path / "paper_2403_11204_amd" / "csrc"
    shutil.copytree(CSRC, csrc)
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    monkeypatch.setattr(bench, "GEMM_TRAFFIC_BYTES_PER_LAUNCH", {4: (1.0e9, bench.product_source_digest())})
    unit = csrc / "gemm.hip"
    text = unit.read_text()
    unit.write_text("// a comment more\n" + text)
    assert bench.gemm_traffic(4) == 1.0e9
    unit.write_text(text.replace("__launch_bounds__(256) void gemm_nt_long_kernel", "__launch_bounds__(512) void gemm_nt_long_kernel"))
    assert bench.gemm_traffic(4) is None
