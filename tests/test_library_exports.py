"""CPU-side checks of the C-ABI library: it loads, exports every symbol the header declares, and its
host-only helpers agree with the paper's printed cost table and with the oracle's size rules."""
import ctypes
import os
import re

import pytest

import oracle

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2511_12280_amd", "libd3tom.so")
HEADER = os.path.join(ROOT, "include", "d3tom.h")


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(LIB):
        from paper_2511_12280_amd import build
        build.build()
    return ctypes.CDLL(LIB)


def test_every_declared_symbol_is_exported(lib):
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    names = sorted(set(re.findall(r"\b(d3tom_[a-z_0-9]+)\s*\(", text)))
    assert {"d3tom_importance", "d3tom_select_topk", "d3tom_merge", "d3tom_attend"} <= set(names)
    for n in names:
        assert hasattr(lib, n), n
    from paper_2511_12280_amd import binding
    assert sorted(binding.EXPORTS) == names
    for n in names:
        assert callable(getattr(binding, n))


def test_host_helpers(lib):
    from paper_2511_12280_amd import binding as B
    for V, r in [(144, 0.25), (1024, 0.10), (3645, 0.10), (3645, 0.5), (10, 0.0), (10, 1.0), (7, 3.0), (2304, 0.3141)]:
        assert B.d3tom_keep_count(V, r) == oracle.keep_count(V, r)
    assert B.d3tom_keep_count(0, 0.5) == 0
    for s in range(32):
        assert B.d3tom_schedule(s, 32, 0.1, 0.5) == pytest.approx(oracle.schedule(s, 32, 0.1, 0.5), abs=1e-15)
    assert B.d3tom_status_string(0) == "ok" and "decider" in B.d3tom_status_string(2)
    for op in range(4):
        assert B.d3tom_workspace_bytes(op, 16, 2688, 2304, 32, 128, 256) >= 256
    assert B.d3tom_workspace_bytes(9, 1, 10, 10, 1, 64, 1) == 0


def test_cost_model_matches_printed_tables(lib):
    from paper_2511_12280_amd import binding as B
    rows = [l.split() for l in open(os.path.join(ROOT, "tests", "golden", "paper_flops_tables.txt"))
            if l.strip() and not l.startswith("#")]
    for src, l_star, alpha, tf in rows:
        got = B.d3tom_model_flops(float(alpha), int(l_star), 32, 32, 1000, 64, 64, 4096, 12288)
        assert round(got / 1e12, 2) == pytest.approx(float(tf), abs=0.0051), (src, l_star, alpha)


def test_device_entry_points_reject_bad_arguments_without_a_gpu(lib):
    # null pointers are refused on the host before anything touches a device
    lib.d3tom_attend.restype = ctypes.c_int
    assert lib.d3tom_attend(None, None, None, 1, 1, None, 1, 1, 64, ctypes.c_float(1.0), None, None, ctypes.c_size_t(0), None) == 1
    lib.d3tom_merge_kv.restype = ctypes.c_int
    i = ctypes.c_int
    assert lib.d3tom_merge_kv(None, None, i(64), i(1), i(1), None, None, None, None, None, None, i(8), i(4), i(2), i(2), i(6),
                              i(0), None, None, None, None, None, None, None, ctypes.c_size_t(0), None) == 1
    f = ctypes.c_float
    for fn in ("d3tom_rmsnorm", "d3tom_rope", "d3tom_linear", "d3tom_stack_step"):
        getattr(lib, fn).restype = ctypes.c_int
    assert lib.d3tom_rmsnorm(None, None, i(4), i(64), f(1e-5), None, None) == 1
    assert lib.d3tom_rope(None, None, None, i(4), i(2), i(64), f(10000.0), None) == 1
    assert lib.d3tom_linear(None, None, i(4), i(64), i(64), i(0), None, None, i(0), None) == 1
    assert lib.d3tom_stack_step(None, i(8), i(256), i(4), i(512), i(1), None, i(1), None, i(0), i(0), i(4), i(2), i(0),
                                f(1e-5), f(10000.0), None, None, None, None, None, None, None, ctypes.c_size_t(0), None) == 1
    lib.d3tom_stack_workspace_bytes.restype = ctypes.c_size_t
    small = lib.d3tom_stack_workspace_bytes(i(208), i(256), i(4), i(512), i(144), i(16))
    big = lib.d3tom_stack_workspace_bytes(i(3773), i(4096), i(32), i(11008), i(3645), i(64))
    assert 0 < small < big < (1 << 30)
    assert lib.d3tom_stack_workspace_bytes(i(0), i(256), i(4), i(512), i(144), i(16)) == 0


def test_stack_step_refuses_a_rotary_base_without_a_gpu(lib):
    # everything else is in order (the addresses are never read on the host, and a refused call enqueues nothing), so a call that
    # is not refused would come back as D3TOM_ERR_DEVICE here
    from paper_2511_12280_amd import binding as B
    i, f, p = ctypes.c_int, ctypes.c_float, ctypes.c_void_p(1 << 20)
    blocks = (ctypes.c_void_p * 6)(*[1 << 20] * 6)
    one = lambda v: (ctypes.c_int32 * 1)(v)
    nbytes = ctypes.c_size_t(B.d3tom_stack_workspace_bytes(48, 256, 4, 512, 40, 2))
    lib.d3tom_stack_step.restype = lib.d3tom_stack_step_batch.restype = ctypes.c_int
    for theta in (1.0, 0.5, 0.0, -1.0, float("nan"), float("inf"), 3.2e38):
        for D in (0, 2):
            assert lib.d3tom_stack_step(p, i(48), i(256), i(4), i(512), i(1), blocks, i(1), p, i(D), i(4), i(40), i(10), i(0), f(1e-5),
                                        f(theta), p, None, None, None, None, None, p, nbytes, None) == 1
            assert lib.d3tom_stack_step_batch(p, i(1), one(48), i(256), i(4), i(512), i(1), blocks, i(1), p, one(D), one(4), one(40), one(10),
                                              i(0), f(1e-5), f(theta), p, None, None, None, None, None, p, nbytes, None) == 1


def test_schedule_variants_share_their_mean(lib):
    from paper_2511_12280_amd import binding as B
    # low -> high (D3ToM-t) and its reverse (D3ToM-t dagger) through the one direction-neutral helper:
    # both are linear between the same two ends, so their mean over the T steps is the midpoint
    # (the calibration the schedule ablation in the appendix states), and they mirror each other
    T, lo, hi = 32, 0.5, 0.9
    fwd = [B.d3tom_schedule(s, T, lo, hi) for s in range(T)]
    rev = [B.d3tom_schedule(s, T, hi, lo) for s in range(T)]
    assert fwd[0] == lo and fwd[-1] == pytest.approx(hi) and all(b > a for a, b in zip(fwd, fwd[1:]))
    assert sum(fwd) / T == pytest.approx((lo + hi) / 2) and sum(rev) / T == pytest.approx((lo + hi) / 2)
    assert rev == pytest.approx(fwd[::-1])



def test_native_binding_refuses_what_it_cannot_pass_on(lib):
    # argument count, tensors that are not on the GPU, addresses in a tensor's place, a float for an int: refused before the
    # library is called; None reaches it as a null pointer and an int as its low 32 bits (status 1: invalid argument)
    import torch
    from paper_2511_12280_amd import _native
    t = torch.zeros(4, 64)
    class Sub(torch.Tensor):
        pass
    assert _native.d3tom_rmsnorm(None, None, 4, 64, 1e-5, None, None) == 1
    assert _native.d3tom_rmsnorm(None, None, 4 + (1 << 32), -64, 1, None, 0) == 1
    with pytest.raises(TypeError):
        _native.d3tom_rmsnorm(None, None, 4, 64, 1e-5, None)
    for bad in (t, t.t(), t.as_subclass(Sub), torch.nn.Parameter(t)):
        with pytest.raises(ValueError, match="contiguous tensors on the GPU"):
            _native.d3tom_rmsnorm(bad, None, 4, 64, 1e-5, None, None)
    for bad in (4096, 0.5, "x"):
        with pytest.raises(AttributeError):
            _native.d3tom_rmsnorm(bad, None, 4, 64, 1e-5, None, None)
    with pytest.raises(TypeError):
        _native.d3tom_rmsnorm(None, None, 4.0, 64, 1e-5, None, None)
    with pytest.raises(TypeError):
        _native.d3tom_rmsnorm(None, None, 4, 64, 1e-5, None, t)


def _kernels(path):
    """Metadata of the gfx950 kernels in the library: the notes of the ELF images inside it."""
    import struct

    import msgpack
    data = open(path, "rb").read()
    kernels, at = [], 0
    while (at := data.find(b"\x7fELF", at + 1)) >= 0:
        if struct.unpack_from("<H", data, at + 18)[0] != 224:              # EM_AMDGPU
            continue
        sh_off, = struct.unpack_from("<Q", data, at + 40)
        sh_size, sh_num = struct.unpack_from("<HH", data, at + 58)
        for i in range(sh_num):
            kind, _, _, off, size = struct.unpack_from("<IQQQQ", data, at + sh_off + i * sh_size + 4)
            if kind == 7:                                                  # SHT_NOTE: name size, description size, type
                names, desc, _ = struct.unpack_from("<III", data, at + off)
                first = at + off + 12 + (names + 3) // 4 * 4
                kernels += msgpack.unpackb(data[first:first + desc])["amdhsa.kernels"]
    return kernels


def test_no_kernel_spills_vector_registers(lib):
    pytest.importorskip("msgpack")
    kernels = _kernels(LIB)
    assert len(kernels) > 100
    spilled = [(k[".name"], k[".vgpr_spill_count"], k[".private_segment_fixed_size"]) for k in kernels
               if k[".vgpr_spill_count"] or k[".private_segment_fixed_size"]]
    assert not spilled, spilled


def test_projection_tiles_are_all_taken(lib):
    """Every tile that is built for a use is the estimate's choice there for some sizes, and no other tile is."""
    import random
    from paper_2511_12280_amd import binding as B
    rng, whole, sliced = random.Random(1), set(), set()
    log_int = lambda lo, hi: int(lo * (hi / lo) ** rng.random())
    for _ in range(20000):
        rows, cols, K = log_int(1, 12000), 8 * log_int(8, 3500), 64 * log_int(1, 220)
        room = 4 * 64 * 256 * 128 if cols <= 8192 else 0
        first, lead, second, slices = B.d3tom_linear_plan(rows, cols, K, room)
        assert 0 < lead <= cols and (lead < cols) == (second >= 0) and (slices == 1 or (K % (64 * slices) == 0 and rows * cols * slices <= room))
        (sliced if slices > 1 else whole).add(B.d3tom_linear_tile_name(first))
    assert sliced == {"64x64 loaders", "64x96 loaders", "64x128 loaders", "96x128 loaders", "128x128", "160x128 loaders", "192x128 loaders", "256x128"}
    assert whole == {"64x64 loaders", "64x96 loaders", "64x128 loaders", "96x128 loaders", "128x128", "128x192 loaders", "128x256",
                     "160x128 loaders", "160x256", "192x128 loaders", "192x256", "224x256", "256x128 loaders", "256x192", "256x256"}


@pytest.mark.parametrize("H,dh,longest,batch", [(32, 128, 8, 9), (32, 128, 32, 16), (8, 128, 200, 9), (32, 128, 65, 8), (32, 64, 65, 16), (16, 64, 200, 9), (32, 64, 32, 1),
                                                (32, 128, 493, 1), (32, 128, 231, 1)])
def test_short_samples_share_the_units(lib, H, dh, longest, batch):
    """Workgroups of 32 queries of the short-sample kernel: two with heads of 128 and four with heads of 64 fit into a unit's 160 KB of LDS, and a batch, of which
    the host knows the longest sample only, takes them always; one long sample whose 64-query tiles fill the units takes those."""
    pytest.importorskip("msgpack")
    from paper_2511_12280_amd import binding as B
    kernel, queries, turns, lds = B.d3tom_attend_plan(B.D3TOM_BF16, batch, longest, H, dh)
    assert (kernel, queries, turns) == (1, 64 if longest == 493 else 32, 0)
    fixed = max(k[".group_segment_fixed_size"] for k in _kernels(LIB) if re.search(rf"attend_bf16_short_kernelILi{dh}ELb[01]ELi{queries // 32}E", k[".name"]))
    assert 1024 <= fixed and (queries == 64 or (lds + fixed) * (2 if dh == 128 else 4) <= 160 * 1024)


@pytest.mark.parametrize("H,lens,dh,form", [
    # tiles of 192 queries (256 with heads of 64) that fill one round of the card's 256 units, and of some XCD's 32 more than one
    (12, [3227], 128, "tiles 256"), (20, [2135], 128, "tiles 256"), (28, [1710], 128, "tiles 256"), (36, [1236], 128, "tiles 256"), (4, [3089] * 3, 128, "tiles 256"),
    (36, [3870], 128, "tiles 256 in turn"), (20, [2687], 64, "tiles 128"),
    (16, [2200], 128, "tiles 192"), (24, [1900], 128, "tiles 192"), (32, [1100], 128, "tiles 192"), (32, [700, 700], 128, "tiles 192"),
    (40, [1538], 128, "tiles 128 in turn"), (48, [1282], 128, "tiles 128 in turn"), (24, [2690], 128, "tiles 192 in turn"),      # last tiles that fit beside the others, or not
    (12, [834, 738, 350], 128, "tiles 128"), (6, [1689, 1200, 900], 128, "tiles 128"),      # batches of which not every sample need have as many tiles as the longest
    (32, [1024], 128, "tiles 128"), (32, [1600], 128, "tiles 256"), (32, [3773], 128, "tiles 256 in turn"), (16, [3500], 64, "tiles 256"),
])
def test_attention_counts_rounds_of_an_xcd(lib, H, lens, dh, form):
    """The width of one sample's query tiles, and whether a batch has tiles of 192, goes by rounds over the 32 units of the XCD with the most heads."""
    from parity import attend_form
    assert attend_form(H, lens, dh) == form
