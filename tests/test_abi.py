"""The C-ABI library loads and exports every symbol include/grass.h declares;
host-side argument checks answer without touching a GPU (CPU only)."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "grass.h")


def _declared_functions():
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    names = re.findall(r"^(?:grass_status|const char\*|int|void)\s+(\w+)\s*\(", text, flags=re.M)
    return sorted(set(names))


@pytest.fixture(scope="module")
def lib():
    from paper_2505_18976_amd import binding
    if not os.path.exists(binding.LIB_PATH):
        import __graft_entry__
        __graft_entry__.build()
    return binding.load_library()


def test_header_declares_the_four_entry_points():
    names = _declared_functions()
    for required in ("grass_mask", "grass_sjlt", "factgrass_linear", "grass_score"):
        assert required in names


def test_every_declared_symbol_is_exported_and_bound(lib):
    from paper_2505_18976_amd import binding
    declared = _declared_functions()
    assert declared == sorted(binding.SIGNATURES)
    for name in declared:
        assert getattr(lib, name) is not None


def test_version_and_strerror(lib):
    assert lib.grass_version() >= 100
    assert lib.grass_strerror(0) == b"ok"
    assert b"invalid" in lib.grass_strerror(1)
    assert b"unknown" in lib.grass_strerror(99)


def test_workspace_queries_validate_on_the_host(lib):
    from paper_2505_18976_amd import binding as b
    out = ctypes.c_size_t(123)
    assert lib.grass_sjlt_workspace_bytes(16, 1000, 0, 64, 1, None, ctypes.byref(out)) == b.GRASS_OK
    assert lib.grass_sjlt_workspace_bytes(16, 1000, 0, 0, 1, None, ctypes.byref(out)) == b.GRASS_EINVAL      # k = 0
    assert lib.grass_sjlt_workspace_bytes(16, 1000, 0, 64, 0, None, ctypes.byref(out)) == b.GRASS_EINVAL     # s = 0
    assert lib.grass_sjlt_workspace_bytes(16, 1000, 0, 64, 3, None, ctypes.byref(out)) == b.GRASS_EINVAL     # s does not divide k
    assert lib.grass_sjlt_workspace_bytes(16, 1000, 2000, 64, 1, None, ctypes.byref(out)) == b.GRASS_EINVAL  # k' > p
    assert lib.grass_sjlt_workspace_bytes(16, 1000, 0, 1 << 20, 1, None, ctypes.byref(out)) == b.GRASS_EUNSUPPORTED
    assert lib.grass_sjlt_workspace_bytes(16, 1000, 0, 64, 1, None, None) == b.GRASS_EINVAL
    assert lib.grass_mask_indices_workspace_bytes(1000, 10, ctypes.byref(out)) == b.GRASS_OK
    assert out.value > 4 * 65536 * 4
    assert lib.grass_mask_indices_workspace_bytes(1000, 1001, ctypes.byref(out)) == b.GRASS_EINVAL
    assert lib.grass_mask_indices_workspace_bytes(1 << 31, 10, ctypes.byref(out)) == b.GRASS_EINVAL
    assert lib.factgrass_linear_workspace_bytes(8, 128, 64, 64, 1024, 1, None, ctypes.byref(out)) == b.GRASS_OK
    assert lib.factgrass_linear_workspace_bytes(8, 128, 64, 129, 1024, 1, None, ctypes.byref(out)) == b.GRASS_EUNSUPPORTED
    assert lib.factgrass_linear_workspace_bytes(8, 0, 64, 64, 1024, 1, None, ctypes.byref(out)) == b.GRASS_EINVAL


@pytest.mark.parametrize("n, m, p", [(1000, 100, 1_863_690), (200, 100, 300_001), (40, 3, 50)])
def test_selective_mask_workspace_holds_what_a_step_uses(lib, n, m, p):
    """The weighted test gradients, at whose place the backward product works later, two matrices of scores, up to 64 partial sums
    of them where they have few tiles, and a sum per 256 columns and per test row; no block beside these."""
    from paper_2505_18976_amd import binding as b
    out = ctypes.c_size_t(0)
    assert lib.grass_selective_mask_grad_workspace_bytes(n, m, p, ctypes.byref(out)) == b.GRASS_OK
    gradients, scores, sums = m * ((p + 3) // 4 * 4) * 4, m * ((n + 15) // 16 * 16) * 4, m * 8 + (p + 255) // 256 * 8
    partial = 64 * m * n * 4 if n * m < 256 * 128 * 256 else 0
    assert gradients + 2 * scores + sums <= out.value <= gradients + 2 * scores + sums + partial + 6 * 256


def test_bad_arguments_are_rejected_before_any_launch(lib):
    """These calls must return on the host: this process has no GPU."""
    from paper_2505_18976_amd import binding as b
    null = ctypes.c_void_p(0)
    fake = ctypes.c_void_p(4096)
    # null pointers
    assert lib.grass_sjlt(null, 4, 100, 100, null, 0, 16, 1, 0, 1, fake, 16, null, 0, None, null) == b.GRASS_EINVAL
    # leading dimension smaller than the row
    assert lib.grass_sjlt(fake, 4, 100, 99, null, 0, 16, 1, 0, 1, fake, 16, null, 0, None, null) == b.GRASS_EINVAL
    assert lib.grass_sjlt(fake, 4, 100, 100, null, 0, 16, 1, 0, 1, fake, 15, null, 0, None, null) == b.GRASS_EINVAL
    # n = 0 is a no-op
    assert lib.grass_sjlt(fake, 0, 100, 100, null, 0, 16, 1, 0, 1, fake, 16, null, 0, None, null) == b.GRASS_OK
    assert lib.grass_mask(fake, 0, 100, 100, fake, 10, fake, 10, null) == b.GRASS_OK
    assert lib.grass_mask(fake, 4, 100, 100, fake, 101, fake, 101, null) == b.GRASS_EINVAL
    assert lib.grass_mask(fake, 4, 100, 100, null, 10, fake, 10, null) == b.GRASS_EINVAL
    # workspace required but missing: many chunks for a single long row
    assert lib.grass_sjlt(fake, 1, 1 << 22, 1 << 22, null, 0, 16, 1, 0, 1, fake, 16, null, 0, None, null) == b.GRASS_EWORKSPACE
    assert lib.grass_mask_indices(0, 0, 1000, 10, fake, null, 0, null) == b.GRASS_EWORKSPACE
    assert lib.grass_score(fake, fake, 2, 8, 8, 8, 8, 8, fake, 8, null, 0, null) == b.GRASS_EINVAL
    assert lib.grass_score(fake, fake, 0, 8, 8, 8, 7, 8, fake, 8, null, 0, null) == b.GRASS_EINVAL
    assert lib.factgrass_linear(fake, fake, 2, 16, 64, 64, fake, 65, fake, 8, 32, 1, 0, 18, fake, 32, null, 0,
                                None, null) == b.GRASS_EINVAL                                                  # k_in' > d_in
    assert lib.grass_gauss_project(fake, 2, 64, 64, 8, 0, 2, 0, 0, fake, 8, null, 0, null) == b.GRASS_EWORKSPACE


def test_logra_refuses_feature_dimensions_beyond_its_offset_range(lib):
    """logra_linear addresses a tile of 64 rows with 32-bit byte offsets: d_in, d_out above 2^24 are refused on the host."""
    from paper_2505_18976_amd import binding as b
    fake, null = ctypes.c_void_p(4096), ctypes.c_void_p(0)
    big = (1 << 24) + 8
    assert lib.logra_linear(fake, fake, 2, 64, big, 64, fake, 8, fake, 8, fake, 64, fake, 1 << 20, null) == b.GRASS_EUNSUPPORTED
    assert lib.logra_linear(fake, fake, 2, 64, 64, big, fake, 8, fake, 8, fake, 64, fake, 1 << 20, null) == b.GRASS_EUNSUPPORTED
    assert lib.logra_linear(fake, fake, 2, 64, 60, 64, fake, 8, fake, 8, fake, 64, fake, 1 << 20, null) == b.GRASS_EUNSUPPORTED  # d % 8


def test_probe_checks_its_buffers_on_the_host(lib):
    from paper_2505_18976_amd import binding as b
    fake, null = ctypes.c_void_p(4096), ctypes.c_void_p(0)
    assert lib.grass_probe_line_reads(null, 1 << 20, fake, 1, 0, 0, 8, null) == b.GRASS_EINVAL
    assert lib.grass_probe_line_reads(fake, 1 << 20, fake, 100, 1, 0, 8, null) == b.GRASS_EINVAL      # 8*256*16 floats needed
    assert lib.grass_probe_line_reads(fake, 1 << 20, fake, 1, 7, 0, 8, null) == b.GRASS_EINVAL        # no such mode
    assert lib.grass_probe_line_reads(ctypes.c_void_p(4100), 1 << 20, fake, 1, 0, 0, 8, null) == b.GRASS_EUNSUPPORTED


def test_noalloc_entry_point_refuses_oversized_problems_on_the_host(lib):
    """grass_sjlt_noalloc keeps its scratch memory in a fixed 32 MiB buffer inside the library: a problem whose
    partial sums need more is refused before anything touches a GPU (this process has none)."""
    from paper_2505_18976_amd import binding as b
    fake, null = ctypes.c_void_p(4096), ctypes.c_void_p(0)
    # 2 column chunks x 1,024 rows x 8,192 buckets x 4 bytes = 64 MiB
    assert lib.grass_sjlt_noalloc(fake, 1024, 1 << 20, 1 << 20, null, 0, 8192, 1, 0, 1, fake, 8192, null) == b.GRASS_ETOOLARGE
    assert b"scratch" in lib.grass_strerror(b.GRASS_ETOOLARGE)
    assert lib.grass_sjlt_noalloc(null, 4, 100, 100, null, 0, 16, 1, 0, 1, fake, 16, null) == b.GRASS_EINVAL
    assert lib.grass_sjlt_noalloc(fake, 0, 100, 100, null, 0, 16, 1, 0, 1, fake, 16, null) == b.GRASS_OK     # n = 0
    assert lib.grass_sjlt_noalloc(fake, 4, 100, 100, null, 0, 16, 3, 0, 1, fake, 16, null) == b.GRASS_EINVAL  # s does not divide k


@pytest.mark.parametrize("n,p,k,s", [(1012, 2149742, 12077, 1), (1022, 17608759, 12864, 4), (1000, 3000001, 16384, 1)])
def test_batches_that_fill_the_chip_in_groups_need_no_scratch(lib, n, p, k, s):
    """About a thousand rows of odd length, one per workgroup: grouped by their offset inside a line they make 1,024 groups,
    one chunk and no partial sums, so the entry point with the fixed buffer takes them (two chunks would need 97 MB)."""
    from paper_2505_18976_amd import binding as b
    text = ctypes.create_string_buffer(200)
    assert lib.grass_sjlt_describe(None, 0, n, p, p, 0, k, s, 1, None, text, 200) == b.GRASS_OK
    assert " chunks=1 " in text.value.decode()


def test_sjlt_plan_follows_what_bounds_a_launch(lib):
    """Launch shapes of calls that an earlier rule ran on a few workgroups or on rows that share nothing worth sharing
    (time with that rule and with this one, in us)."""
    from paper_2505_18976_amd import binding as b

    def plan(n, p, kp, k, s, bf16):
        text = ctypes.create_string_buffer(200)
        assert lib.grass_sjlt_describe(4096, bf16, n, p, p, kp, k, s, 1, None, text, 200) == b.GRASS_OK
        name, grid, block, _, chunks = text.value.decode().split(" ")[:5]
        return int(name.split(",")[1]), int(block[6:]), int(chunks[7:])
    assert plan(3, 4_359_211, 0, 224, 4, 1)[2] >= 60                       # 201 -> 76: chunks are whole steps of positions
    assert plan(42, 110_868, 110_643, 22_254, 1, 0)[2] >= 2                # 47 -> 28: the work on a position, not its bytes
    assert plan(1_104, 92_347, 0, 232, 4, 0)[0] == 1                       # 450 -> 379: an add per non-zero and row is not shared
    assert plan(1_765, 69_547, 69_547, 189, 1, 0)[0] == 2                  # 145 -> 120: index and hash are
    assert plan(2_895, 17_275, 0, 1_551, 1, 1)[1] == 512                   # 59 -> 45: one pass of 1,024 threads and a bit
    assert plan(3, 57_852, 9_819, 96, 1, 0)[2] == 1                        # 12.8 -> 10.3: a second launch costs the host more


@pytest.mark.parametrize("n,chunks", [(600, 2), (511, 4), (1100, 0)])
def test_sjlt_query_reserves_what_the_call_can_use(lib, n, chunks):
    """511 rows of k = 16,384 are cut into up to four chunks; from 512 on a batch is large and has two at most, from 1,024
    on one and no partial sums."""
    out = ctypes.c_size_t(0)
    assert lib.grass_sjlt_workspace_bytes(n, 2_000_000, 0, 16_384, 4, None, ctypes.byref(out)) == 0
    assert out.value == chunks * n * 16_384 * 4


@pytest.mark.parametrize("n,T,chunks", [(32, 512, 6), (10, 1889, 20), (88, 241, 2), (66, 103, 1), (131, 77, 1), (60, 40, 1),
                                        (127, 130, 2)])
def test_factgrass_chunks(lib, n, T, chunks):
    """Partial sums the query reserves = chunks of a sample.  88 x 241 would be 264 workgroups of 96 tokens (34 us, 26 with
    128) and 131 x 77 262 of 64 and a kernel that adds them (23 us, 15 with whole sequences)."""
    out = ctypes.c_size_t(0)
    layers = 2 if (n, T) == (66, 103) else 1
    if layers == 2:
        assert lib.factgrass_layers_workspace_bytes(2, n, T, 64, 64, 512, 1, None, ctypes.byref(out)) == 0
        assert out.value < 1 << 16
    else:
        assert lib.factgrass_linear_workspace_bytes(n, T, 64, 64, 512, 1, None, ctypes.byref(out)) == 0
        assert out.value == (0 if chunks == 1 else chunks * n * 512 * 4)


def test_tuning_is_a_per_call_argument(lib):
    """Launch-shape overrides travel with the call: the same query with and without them, interleaved, keeps
    answering the same (there is no process-wide setting to leak from one call into the next)."""
    from paper_2505_18976_amd import binding as b
    plain, tuned = ctypes.c_size_t(0), ctypes.c_size_t(0)
    t = b.GrassTuning(sjlt_rows_per_block=1, sjlt_column_chunks=7, sjlt_threads=256, sjlt_accumulator=2)
    for _ in range(2):
        assert lib.grass_sjlt_workspace_bytes(64, 40000, 0, 1024, 1, None, ctypes.byref(plain)) == b.GRASS_OK
        assert lib.grass_sjlt_workspace_bytes(64, 40000, 0, 1024, 1, ctypes.byref(t), ctypes.byref(tuned)) == b.GRASS_OK
        assert tuned.value == 7 * 64 * 1024 * 4 and plain.value != tuned.value
    ft = b.GrassTuning(factgrass_tokens_per_block=64)
    for _ in range(2):
        assert lib.factgrass_linear_workspace_bytes(4, 256, 64, 64, 512, 1, None, ctypes.byref(plain)) == b.GRASS_OK
        assert lib.factgrass_linear_workspace_bytes(4, 256, 64, 64, 512, 1, ctypes.byref(ft), ctypes.byref(tuned)) == b.GRASS_OK
        assert tuned.value == 4 * 4 * 512 * 4 and plain.value != tuned.value
    # a missing workspace is reported for the tuned plan, before any launch
    fake, null = ctypes.c_void_p(4096), ctypes.c_void_p(0)
    assert lib.grass_sjlt(fake, 64, 40000, 40000, null, 0, 1024, 1, 0, 1, fake, 1024, null, 0, ctypes.byref(t),
                          null) == b.GRASS_EWORKSPACE


@pytest.mark.parametrize("stream_id", [0, 18, (1 << 64) - 1, -1, (1 << 64) + 5])
def test_layer_table_takes_stream_ids_modulo_2_64(monkeypatch, stream_id):
    """As every other entry point does with its integers."""
    import torch
    from paper_2505_18976_amd import binding

    class Lib:
        def factgrass_layers(self, table, n_layers, *rest):
            self.table = (binding.FactgrassLayer * n_layers).from_buffer_copy(table)
            return binding.GRASS_OK
    lib = Lib()
    monkeypatch.setattr(binding, "load_library", lambda: lib)
    monkeypatch.setattr(binding, "_stream", lambda: 0)
    x, g = torch.zeros(2, 3, 8, dtype=torch.bfloat16), torch.zeros(2, 3, 16, dtype=torch.bfloat16)
    ii, io = torch.zeros(4, dtype=torch.int32), torch.zeros(5, dtype=torch.int32)
    out = torch.zeros(2, 14)
    binding.factgrass_layers([(x, g, ii, io, 3), (g, x, ii, io, stream_id)], 7, 1, 0, out, ws=torch.zeros(8, dtype=torch.uint8))
    a, b = lib.table
    assert (a.x, a.gout, a.idx_in, a.idx_out, a.d_in, a.d_out, a.stream_id, a.out) == (
        x.data_ptr(), g.data_ptr(), ii.data_ptr(), io.data_ptr(), 8, 16, 3, out.data_ptr())
    assert (b.d_in, b.d_out, b.stream_id, b.out) == (16, 8, stream_id % (1 << 64), out.data_ptr() + 28)


def test_binding_refuses_to_run_without_the_library(monkeypatch, tmp_path):
    from paper_2505_18976_amd import binding
    monkeypatch.setattr(binding, "_lib", None)
    monkeypatch.setattr(binding, "LIB_PATH", str(tmp_path / "missing.so"))
    with pytest.raises(ImportError):
        binding.load_library()
