"""LoGra's two kernels at the edges of their tilings: columns cut into ranges, token tiles that cross samples, samples that
do not fill a group of eight, projected widths that are no multiple of 16, and token chunks that are added by the
workgroup that arrives last (bit-reproducible)."""
import numpy as np
import pytest
import torch

import synth
from oracle import grass_oracle as orc

pytestmark = pytest.mark.gpu
TOL_LOGRA = 1e-4          # exact bf16 products, fp32 sums over d and over tokens: the bar of the other LoGra tests


@pytest.mark.parametrize("n,T,d_in,d_out,ki,ko", [
    (1, 1, 8, 8, 1, 1),
    (3, 43, 72, 56, 17, 33),              # one group and a partial one; a token tile that crosses all samples
    (9, 129, 64, 2_048, 64, 5),           # second group of eight samples; widths 32 : 1
    (2, 100, 4_104, 3_000, 48, 64),       # few tokens: many ranges, ragged last group
    (17, 256, 264, 136, 16, 16),
    (1, 5_000, 128, 200, 64, 64),         # token chunks
    (2, 4_097, 64, 64, 40, 24),
])
def test_logra_ranges_and_chunks(n, T, d_in, d_out, ki, ko):
    import paper_2505_18976_amd as grass
    dev = torch.device("cuda:0")
    x, g = synth.linear_layer_factors(n, T, d_in, d_out, seed=97, device=dev)
    Pi = grass.grass_to_bf16(grass.grass_gauss_matrix(0, 40, d_in, ki, 0, d_in, device=dev))
    Po = grass.grass_to_bf16(grass.grass_gauss_matrix(0, 41, d_out, ko, 0, d_out, device=dev))
    wide = torch.full((n, ki * ko + 3), 7.0, device=dev)
    out = grass.logra_linear(x, g, Pi, Po, out=wide[:, :ki * ko])
    again = [grass.logra_linear(x, g, Pi, Po) for _ in range(3)]
    h = lambda t: t.float().cpu().numpy().astype(np.float64)
    assert orc.max_rel_err(h(out), orc.logra_linear(h(x), h(g), h(Pi), h(Po))) <= TOL_LOGRA
    assert all(torch.equal(a, out) for a in again) and bool((wide[:, ki * ko:] == 7.0).all())


@pytest.mark.parametrize("n,T,d_in,d_out,ki,ko,free", [
    (1, 1, 64, 64, 8, 8, True), (5, 64, 104, 1_000, 64, 64, True), (5, 65, 104, 40, 33, 64, False),
    (345, 24, 112, 48, 64, 64, True), (255, 100, 72, 136, 64, 17, False), (256, 256, 72, 40, 48, 64, True),
    (300, 129, 264, 8, 64, 1, True), (257, 257, 64, 64, 16, 16, False), (70, 33, 3_000, 16, 64, 64, True),
])
def test_logra_in_one_launch_and_without_workspace(n, T, d_in, d_out, ki, ko, free):
    """Short samples run in one launch where that is faster; without a workspace all calls do that never needed one, the others
    are refused."""
    import ctypes
    import paper_2505_18976_amd as grass
    from paper_2505_18976_amd import binding as b
    dev = torch.device("cuda:0")
    x, g = synth.linear_layer_factors(n, T, d_in, d_out, seed=98, device=dev)
    Pi = grass.grass_to_bf16(grass.grass_gauss_matrix(0, 40, d_in, ki, 0, d_in, device=dev))
    Po = grass.grass_to_bf16(grass.grass_gauss_matrix(0, 41, d_out, ko, 0, d_out, device=dev))
    h = lambda t: t.float().cpu().numpy().astype(np.float64)
    ref = orc.logra_linear(h(x), h(g), h(Pi), h(Po))
    assert orc.max_rel_err(h(grass.logra_linear(x, g, Pi, Po)), ref) <= TOL_LOGRA
    out = torch.full((n, ki * ko + 1), 7.0, device=dev)
    null = ctypes.c_void_p(0)
    status = grass.load_library().logra_linear(x.data_ptr(), g.data_ptr(), n, T, d_in, d_out, Pi.data_ptr(), ki, Po.data_ptr(), ko,
                                               out.data_ptr(), ki * ko + 1, null, 0, torch.cuda.current_stream().cuda_stream)
    assert status == (b.GRASS_OK if free else b.GRASS_EWORKSPACE)
    if free:
        assert orc.max_rel_err(h(out[:, :ki * ko]), ref) <= TOL_LOGRA and bool((out[:, ki * ko] == 7.0).all())
    else:
        assert bool((out == 7.0).all())
