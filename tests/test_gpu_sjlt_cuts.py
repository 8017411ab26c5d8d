"""Launches that are cut into column chunks with one or two rows per workgroup: every row at its own offset inside a line,
two rows sharing hashes when they can be grouped by that offset, and the entry point whose scratch memory limits the
number of chunks.  Bar: 1e-5 row-relative, as in the other SJLT tests (sums in fp64, at most 96 fp32 partial sums)."""
import pytest
import torch

import synth
from oracle import grass_oracle as orc

pytestmark = pytest.mark.gpu
TOL = 1e-5


@pytest.mark.parametrize("n,p,kp,k,s,bf16", [
    (1, 32_769, 0, 64, 1, False), (3, 70_001, 0, 100, 1, False), (17, 65_537, 0, 1_000, 1, False),
    (70, 40_001, 0, 96, 4, False),           # two rows per workgroup, a ragged last block of groups
    (63, 40_001, 0, 96, 4, False),           # one row short of grouping
    (130, 40_003, 0, 512, 1, True), (530, 20_001, 0, 64, 1, False), (5, 300_007, 0, 16_384, 1, True),
    (2, 40_000, 0, 20_000, 1, False),        # fp32 buckets
    (7, 100_003, 8_193, 128, 1, False), (300, 60_000, 20_001, 252, 4, True), (513, 30_000, 9_000, 33, 1, False),
    (1_701, 30_000, 20_000, 33, 1, False),   # masked, two rows per workgroup, an odd number of rows
    (1_401, 20_000, 9_001, 64, 1, True),
    (1_025, 6_000, 2_000, 40, 1, False), (2_001, 17_275, 0, 60, 1, True), (1_030, 7_001, 0, 96, 1, False),   # 512 threads
    (3, 1_200_007, 0, 224, 4, True),         # many chunks of whole steps
    (42, 90_001, 90_001, 22_254, 1, False),  # fp32 buckets, every entry kept, chunks
])
def test_cut_launches(n, p, kp, k, s, bf16):
    import paper_2505_18976_amd as grass
    dev = torch.device("cuda:0")
    g = synth.bernoulli_sparse_normal(n, p, 0.3, 1.0, seed=n + p, device=dev)
    g = g.to(torch.bfloat16) if bf16 else g
    idx = grass.grass_mask_indices(5, 0, p, kp, device=dev) if kp else None
    f = grass.grass_sjlt_bf16 if bf16 else grass.grass_sjlt
    out = torch.full((n, k + 1), 7.0, device=dev)
    f(g, k, s, 5, 1, idx=idx, out=out[:, :k])
    assert torch.equal(f(g, k, s, 5, 1, idx=idx), out[:, :k]) or k > 16_384      # fp32 buckets add in any order
    rows = sorted({0, 1 % n, n // 2, n - 1})
    gh = g[rows].float().cpu().numpy()
    ref = orc.grass(gh, idx.cpu().numpy(), k, s, 5, 1) if kp else orc.sjlt(gh, k, s, 5, 1)
    assert orc.max_rel_err(out[rows][:, :k].cpu().numpy(), ref) <= TOL and bool((out[:, k] == 7.0).all())


def test_fixed_scratch_limits_the_chunks():
    """100 rows x 8,192 sums: 20 chunks would take 65 MB of partial sums, the fixed buffer holds 10."""
    import paper_2505_18976_amd as grass
    dev = torch.device("cuda:0")
    g = synth.bernoulli_sparse_normal(100, 400_001, 0.3, 1.0, seed=9, device=dev)
    out = torch.empty((100, 8_192), device=dev)
    grass.grass_sjlt_noalloc(g, 8_192, 1, 5, 1, out)
    ref = orc.sjlt(g[[0, 99]].cpu().numpy(), 8_192, 1, 5, 1)
    assert orc.max_rel_err(out[[0, 99]].cpu().numpy(), ref) <= TOL


@pytest.mark.parametrize("n,p,kp,k,s,bf16,free", [
    (2, 118_046, 0, 14_076, 4, False, True), (3, 24_051, 16_195, 49, 1, False, True), (8, 27_147, 27_147, 1_451, 1, True, True),
    (7, 123_835, 0, 23_666, 1, False, True), (21, 80_117, 0, 7_172, 4, True, True),
    (6, 31_000, 31_000, 64, 1, False, True),
    (1, 1 << 20, 0, 16, 1, False, False),
])
def test_calls_that_never_needed_a_workspace(n, p, kp, k, s, bf16, free):
    """Without a workspace a call that would be cut into chunks runs uncut if that needs none, and is refused otherwise."""
    import ctypes
    import paper_2505_18976_amd as grass
    from paper_2505_18976_amd import binding as b
    dev = torch.device("cuda:0")
    g = synth.bernoulli_sparse_normal(n, p, 0.3, 1.0, seed=n + p, device=dev)
    g = g.to(torch.bfloat16) if bf16 else g
    idx = grass.grass_mask_indices(5, 0, p, kp, device=dev) if kp else None
    out = torch.full((n, k), 7.0, device=dev)
    f = grass.load_library().grass_sjlt_bf16 if bf16 else grass.load_library().grass_sjlt
    status = f(g.data_ptr(), n, p, p, idx.data_ptr() if kp else None, kp, k, s, 5, 1, out.data_ptr(), k, ctypes.c_void_p(0), 0, None,
               torch.cuda.current_stream().cuda_stream)
    assert status == (b.GRASS_OK if free else b.GRASS_EWORKSPACE)
    if not free:
        assert bool((out == 7.0).all())
        return
    gh = g.float().cpu().numpy()
    ref = orc.grass(gh, idx.cpu().numpy(), k, s, 5, 1) if kp else orc.sjlt(gh, k, s, 5, 1)
    assert orc.max_rel_err(out.cpu().numpy(), ref) <= TOL
