"""Registers and scratch of the built kernels, as the compiler reported them
(paper_2608_27888_amd/libntc.kernels.json, written by the build): the launch shapes
count on the occupancy, and a spilled register is memory traffic inside a loop."""
import json
import re

import pytest

from paper_2608_27888_amd import build


@pytest.fixture(scope="module")
def kernels():
    with open(build.KERNELS) as f:
        return {name: used for per in json.load(f).values() for name, used in per.items()}


def named(kernels, part):
    found = {k: v for k, v in kernels.items() if part in k}
    assert found, part
    return found


def test_report_is_read_whole():
    report = """a.hip:3:1: warning: real [-Wsome]
    3 | code
      | ^
In file included from b.hip:2:
c.h:7:1: remark: Function Name: _Zk [-Rpass-analysis=kernel-resource-usage]
    7 | __global__
      | ^
In file included from b.hip:2:
c.h:7:1: remark:     VGPRs: 57 [-Rpass-analysis=kernel-resource-usage]
    7 | __global__
      | ^
c.h:7:1: remark:     ScratchSize [bytes/lane]: 8 [-Rpass-analysis=kernel-resource-usage]
    7 | __global__
      | ^
c.h:7:1: remark:     Dynamic Stack: False [-Rpass-analysis=kernel-resource-usage]
    7 | __global__
      | ^
In file included from b.hip:2:
c.h:9:1: warning: other [-Wsome]"""
    used, rest = build.resources(report)
    assert used == {"_Zk": {"VGPRs": 57, "ScratchSize": 8}}
    assert rest == ["a.hip:3:1: warning: real [-Wsome]", "    3 | code", "      | ^",
                    "In file included from b.hip:2:", "c.h:9:1: warning: other [-Wsome]"]


def test_binning_runs_eight_waves_a_simd_without_scratch(kernels):
    """Two 16-wave workgroups a CU need eight waves a SIMD: at most 64 registers."""
    for part in ("bins_count", "bins_place"):
        for name, used in named(kernels, part).items():
            assert used["ScratchSize"] == 0, (name, used)
            assert used["VGPRs"] <= 64, (name, used)
            assert used["Occupancy"] == 8, (name, used)


def decode(kernels, kernel, **shape):
    """Decode kernels by their template arguments."""
    pattern = re.compile(kernel + r"ILi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELb(\d)ELi(\d)ELb(\d)E")
    names = ("levels", "channels", "pe", "hidden", "hidden_layers", "mip", "store", "leaky")
    found = {}
    for k, v in kernels.items():
        m = pattern.search(k)
        if m:
            args = dict(zip(names, map(int, m.groups())))
            if all(args[n] == want for n, want in shape.items()):
                found[k] = (args, v)
    assert found, (kernel, shape)
    return found


def test_binned_decode_of_64_wide_runs_four_waves_a_simd(kernels):
    """Two waves a SIMD were slower on most shapes.  At four, decoders with two hidden
    layers or a positional encoding may spill a little; the plain ones may not."""
    for name, (args, used) in decode(kernels, "decode_binned", hidden=64).items():
        assert used["Occupancy"] >= 4, (name, used)
        assert used["ScratchSize"] <= 64, (name, used)
        if args["hidden_layers"] == 1 and args["pe"] == 0 and args["levels"] == 2:
            assert used["ScratchSize"] == 0, (name, used)


def test_stream_decode_of_64_wide_holds_its_weights(kernels):
    """No scratch beside the weights in registers, but for the largest decoder (3 x 16
    channels, two hidden layers, 26 fragments) and one store form of 2 x 8 channels
    with 8 octaves."""
    for name, (args, used) in decode(kernels, "decode_stream_reg", hidden=64).items():
        largest = args["levels"] == 3 and args["hidden_layers"] == 2
        octaves = args["channels"] == 8 and args["pe"] == 32
        assert used["ScratchSize"] <= (52 if largest else 8 if octaves else 0), (name, used)
