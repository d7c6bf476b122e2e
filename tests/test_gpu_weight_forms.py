"""GPU parity of the decode where its weight forms, workgroup widths and tile deals
change: weights in registers (64-wide, stream order) or in LDS, taps ahead of the
MLP or gathered in place, decoder blocks at odd offsets (an odd output width), calls
that fill a fraction of the chip up to several tiles per wave, and non-finite latents.

Tolerance 2e-3 (max-abs on channels in [0, 1]): fp16 operands and activations,
fp32 accumulation, as everywhere in the decode tests.
"""
import sys

import numpy as np
import pytest
import torch

from paper_2608_27888_amd import ntc
from paper_2608_27888_amd import workloads as W

pytestmark = pytest.mark.gpu

TOL = 2e-3


@pytest.fixture(scope="module")
def dev():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    ntc.lib()
    return torch.device("cuda:0")


def workload(seed, n, levels, ch, hid, nh, out, octaves, mip, T=11, D=5):
    rng = np.random.default_rng(seed)
    res = [24, 12, 6][:levels]
    dims = [levels * ch + 4 * octaves] + [hid] * (1 + nh) + [out]
    runs = rng.integers(1, 200, n // 40 + 2)  # screen-coherent runs of one texture
    tex = np.repeat(rng.integers(0, T, runs.size), runs)[:n]
    tex = np.concatenate([tex, rng.integers(0, T, n - tex.size)]).astype(np.uint32)
    uv = rng.random((n, 2), dtype=np.float32)
    return W.Workload("forms", T, res, [ch] * levels, W.draw_latents(seed, T, res, [ch] * levels),
                      D, dims, W.draw_decoders(seed, D, dims), (np.arange(T) % D).astype(np.uint32),
                      tex, uv, rng.uniform(0, levels, n).astype(np.float32) if mip else None,
                      None, {}, octaves)


def both(dev, w):
    model, q = ntc.upload(w, dev)
    bins = ntc.build_bins(q.tex_id, model.tex_to_dec, w.n_decoders)
    a, b = ntc.decode(model, q, bins), ntc.decode(model, q)
    assert torch.equal(a.view(torch.int32), b.view(torch.int32)), "binned and stream bits differ"
    return a


@pytest.mark.parametrize("levels,ch,hid,nh,out,octaves,mip", [
    (2, 8, 64, 1, 8, 0, False),      # 14 fragments, layer 0 half padded
    (2, 16, 64, 1, 7, 0, False),     # odd blocks: 2-byte aligned fragment loads
    (2, 16, 64, 1, 16, 4, False),    # 18 fragments, wide rows
    (2, 16, 64, 1, 9, 8, False),
    (2, 16, 64, 2, 5, 0, False),     # 22 fragments: gathered in place
    (3, 16, 64, 1, 8, 0, False),     # 48 features: the second K-step half padded
    (3, 16, 64, 2, 3, 0, True),      # 26 fragments
    (2, 16, 64, 1, 1, 0, True),
    (2, 8, 128, 1, 11, 0, False),    # weights in LDS, odd blocks
    (3, 16, 128, 2, 8, 0, True),
])
def test_weight_forms(dev, oracle, levels, ch, hid, nh, out, octaves, mip):
    w = workload(3, 9001, levels, ch, hid, nh, out, octaves, mip)
    print(f"[forms] {levels}x{ch} dims={w.dims} mip={mip}", file=sys.stderr, flush=True)
    assert np.abs(both(dev, w).cpu().numpy() - oracle.decode(w)).max() <= TOL


@pytest.mark.parametrize("tiles", [1, 3, 255, 256, 257, 513, 1025, 2049, 8 * 1024 + 9])
@pytest.mark.parametrize("D", [1, 3, 70])
def test_workgroup_widths_and_deal(dev, oracle, tiles, D):
    """Around the tile counts where the stream decode's workgroups get wider, up to
    several tiles a wave, with one decoder, few, and more than one probe round of the
    bin search."""
    n = tiles * 64 - 17
    w = workload(tiles + D, n, 2, 8, 64, 1, 4, 0, False, T=80, D=D)
    print(f"[deal] n={n} D={D}", file=sys.stderr, flush=True)
    got = both(dev, w).cpu().numpy()
    pick = np.unique(np.linspace(0, n - 1, min(n, 4000)).astype(np.int64))
    part = W.Workload("part", w.n_textures, w.res, w.channels, w.latents, D, w.dims, w.params,
                      w.tex_to_dec, w.tex_id[pick].copy(), w.uv[pick].copy(), None)
    assert np.abs(got[pick] - oracle.decode(part)).max() <= TOL


@pytest.mark.parametrize("tiles", [4090, 4096, 4099, 8197])
@pytest.mark.parametrize("D,T,nh,mip", [(1, 1, 1, False), (40, 7, 1, True), (9, 9, 2, False)])
def test_binned_ranges_of_two_workgroups_a_cu(dev, oracle, tiles, D, T, nh, mip):
    """Around the size from which every CU has two full workgroups, whose ranges of
    tiles are then unequal: every row written once, with the stream decode's bits,
    over bins without queries (7 textures of 40 decoders) too."""
    n = tiles * 64 - 13
    w = workload(tiles + D, n, 2, 16, 64, nh, 8, 0, mip, T=T, D=D)
    print(f"[two-groups] tiles={tiles} D={D} nh={nh} mip={mip}", file=sys.stderr, flush=True)
    got = both(dev, w).cpu().numpy()
    pick = np.unique(np.linspace(0, n - 1, 4000).astype(np.int64))
    part = W.Workload("part", w.n_textures, w.res, w.channels, w.latents, D, w.dims, w.params,
                      w.tex_to_dec, w.tex_id[pick].copy(), w.uv[pick].copy(),
                      w.mip[pick].copy() if mip else None)
    assert np.abs(got[pick] - oracle.decode(part)).max() <= TOL


@pytest.mark.parametrize("levels,ch,nh,out,octaves,mip", [
    (2, 16, 1, 7, 4, False),     # 18 fragments: 8 cached decoders
    (3, 16, 2, 3, 0, True),      # 26 fragments: 5
])
@pytest.mark.parametrize("D", [4, 40])
def test_stream_decoder_cache(dev, oracle, levels, ch, nh, out, octaves, mip, D):
    """A stream long enough for the workgroups' decoder cache, with fewer decoders
    than it holds and with more (slots shared by several, filled by one)."""
    n = 1025 * 64 + 5
    w = workload(50 + D, n, levels, ch, 64, nh, out, octaves, mip, T=60, D=D)
    print(f"[cache] dims={w.dims} D={D}", file=sys.stderr, flush=True)
    got = both(dev, w).cpu().numpy()
    pick = np.unique(np.linspace(0, n - 1, 4000).astype(np.int64))
    part = W.Workload("part", w.n_textures, w.res, w.channels, w.latents, D, w.dims, w.params,
                      w.tex_to_dec, w.tex_id[pick].copy(), w.uv[pick].copy(),
                      None if w.mip is None else w.mip[pick].copy(), None, {}, octaves)
    assert np.abs(got[pick] - oracle.decode(part)).max() <= TOL


@pytest.mark.parametrize("hid", [64, 128])
def test_non_finite_latents_stay_in_their_queries(dev, hid):
    """Infinities, NaN and overflowing activations of one texture change no row of
    another's queries, though they share tiles and MFMAs."""
    w = workload(8, 20000, 2, 16, hid, 1, 8, 0, False, D=1)
    clean = both(dev, w)
    lat = w.latents.reshape(w.n_textures, -1).copy()
    lat[4, ::3], lat[4, 1::3], lat[4, 2::3] = 0x7C00, 0x7E00, 0x7BFF  # inf, NaN, 65504
    w.latents = lat.reshape(-1)
    print(f"[non-finite] hid={hid}", file=sys.stderr, flush=True)
    got = both(dev, w)
    other = torch.from_numpy(w.tex_id != 4).to(dev)
    assert torch.equal(got[other], clean[other])
