"""GPU parity of the blocks around the merge layer and of the whole denoising step (Algorithm 1's loop
over layers) against the fp64 oracle in oracle/stack.py, through the C ABI.

Tolerances.  Every stored tensor is bf16 on both sides, rounded once from a float32 (GPU) or float64
(oracle) value.  For a single operation fed with identical inputs the two roundings can differ by one
bf16 step (2^-8 relative in the worst binade position) when the exact value sits next to a rounding
boundary, plus the float32 accumulation error of the GPU (<= K * 2^-24 relative to the sum of magnitudes).
So the single-operation bound is |gpu - ref| <= 2^-7 |ref| + 1e-3 * rms(ref) ("one step").  Through a whole
stack such one-step differences feed later layers; the bound there is on the relative rms difference and
on the largest absolute difference, stated with each test.
"""
import numpy as np
import pytest
import torch

import oracle
from oracle import stack as OS
from paper_2511_12280_amd import workloads as W
import parity as P
from stack_chain import jittered_bf16, stack_step_given

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2511_12280_amd import binding
    assert torch.cuda.is_available(), "GPU tests need a device"
    return binding


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to("cuda").to(torch.bfloat16).contiguous()


def _host(t):
    return t.detach().to(torch.float32).cpu().numpy().astype(np.float64)


def _one_step(got, ref, what):
    ref = np.asarray(ref, dtype=np.float64)
    rms = np.sqrt(np.mean(ref * ref)) + 1e-30
    excess = np.abs(got - ref) - (2.0 ** -7 * np.abs(ref) + 1e-3 * rms)
    assert excess.max() <= 0, f"{what}: {np.abs(got - ref).max():.3e} abs, worst excess {excess.max():.3e}"
    # and nearly all elements agree exactly (same rounding of nearly the same number)
    same = np.mean(got == ref)
    assert same > 0.97, f"{what}: only {same:.3f} of the elements are bit-identical"


# ---- RMSNorm -----------------------------------------------------------------------------------
@pytest.mark.parametrize("rows,d", [(1, 8), (37, 256), (5, 1032), (130, 4096), (3, 8192)])
def test_rmsnorm(B, rows, d):
    rng = np.random.default_rng([rows, d])
    x = W.round_to((rng.standard_normal((rows, d)) * rng.uniform(0.1, 30.0, (rows, 1))).astype(np.float32), "bf16")
    g = W.round_to((1.0 + 0.3 * rng.standard_normal(d)).astype(np.float32), "bf16")
    y = torch.empty(rows, d, dtype=torch.bfloat16, device="cuda")
    B.d3tom_rmsnorm(_dev(x), _dev(g), 1e-5, y)
    torch.cuda.synchronize()
    _one_step(_host(y), OS.round_bf16(OS.rmsnorm(x, g, 1e-5)), "rmsnorm")


def test_rmsnorm_in_place(B):
    rng = np.random.default_rng(3)
    x = W.round_to(rng.standard_normal((50, 512)).astype(np.float32), "bf16")
    g = W.round_to((1.0 + 0.3 * rng.standard_normal(512)).astype(np.float32), "bf16")
    t = _dev(x)
    B.d3tom_rmsnorm(t, _dev(g), 1e-6, t)
    torch.cuda.synchronize()
    _one_step(_host(t), OS.round_bf16(OS.rmsnorm(x, g, 1e-6)), "rmsnorm in place")


def test_rmsnorm_rejects(B):
    x = torch.zeros(4, 12, dtype=torch.bfloat16, device="cuda")
    g = torch.ones(12, dtype=torch.bfloat16, device="cuda")
    with pytest.raises(B.D3tomError) as e:
        B.d3tom_rmsnorm(x, g, 1e-5, x)
    assert e.value.status == B.D3TOM_ERR_UNSUPPORTED          # row length not a multiple of 8
    x = torch.zeros(4, 16, dtype=torch.bfloat16, device="cuda")
    with pytest.raises(B.D3tomError) as e:
        B.d3tom_rmsnorm(x, torch.ones(16, dtype=torch.bfloat16, device="cuda"), -1.0, x)
    assert e.value.status == B.D3TOM_ERR_INVALID_ARG


# ---- rotary embedding --------------------------------------------------------------------------
@pytest.mark.parametrize("rows,H,dh,theta", [(9, 3, 64, 10000.0), (300, 2, 128, 10000.0), (17, 32, 128, 500000.0),
                                             (4, 1, 16, 10000.0), (6, 2, 256, 10000.0)])
def test_rope(B, rows, H, dh, theta):
    rng = np.random.default_rng([rows, H, dh])
    q = W.round_to(rng.standard_normal((rows, H, dh)).astype(np.float32), "bf16")
    k = W.round_to(rng.standard_normal((rows, H, dh)).astype(np.float32), "bf16")
    pos = np.sort(rng.choice(3773, size=rows, replace=False)).astype(np.int32)
    pos[0] = 0; pos[-1] = 3772
    tq, tk = _dev(q), _dev(k)
    B.d3tom_rope(tq, tk, torch.from_numpy(pos).cuda(), theta)
    torch.cuda.synchronize()
    _one_step(_host(tq), OS.round_bf16(OS.rope(q, pos, theta)), "rope q")
    _one_step(_host(tk), OS.round_bf16(OS.rope(k, pos, theta)), "rope k")
    np.testing.assert_array_equal(_host(tq)[0], q[0].astype(np.float64))       # position 0 is the identity


# ---- projections -------------------------------------------------------------------------------
def _linear_tiles():
    if not torch.cuda.is_available():                  # collected without a GPU too, where the library may not be built yet
        return []
    from paper_2511_12280_amd import binding
    names = []
    while (name := binding.d3tom_linear_tile_name(len(names))) is not None:
        names.append(name)
    return names


LIN_TILES = _linear_tiles()


def _chosen(M, N, K):
    from paper_2511_12280_amd import binding
    first, cols, second, slices = binding.d3tom_linear_plan(M, N, K)
    assert slices == 1 and (cols == N) == (second < 0)
    return LIN_TILES[first] + (" + " + LIN_TILES[second] if second >= 0 else "")


LIN_SHAPES = [(1, 8, 64), (5, 128, 64), (64, 128, 128), (200, 384, 256), (493, 512, 1024), (129, 200, 64), (300, 1000, 192),
              (1000, 256, 4096)]


@pytest.mark.parametrize("tile", [1, 2, 4])
@pytest.mark.parametrize("M,N,K", LIN_SHAPES)
def test_linear_plain_and_residual(B, M, N, K, tile):
    rng = np.random.default_rng([M, N, K])
    a = W.round_to(rng.standard_normal((M, K)).astype(np.float32), "bf16")
    w = W.round_to((rng.standard_normal((N, K)) / np.sqrt(K)).astype(np.float32), "bf16")
    r = W.round_to(rng.standard_normal((M, N)).astype(np.float32), "bf16")
    ref = OS.linear(a, w)
    ta, tw, tr = _dev(a), _dev(w), _dev(r)
    out = torch.full((M, N), 7.0, dtype=torch.bfloat16, device="cuda")
    B.d3tom_linear_tile(ta, tw, B.D3TOM_LINEAR_PLAIN, out, tile)
    torch.cuda.synchronize()
    _one_step(_host(out), OS.round_bf16(ref), f"plain {M}x{N}x{K} tile {tile}")
    B.d3tom_linear_tile(ta, tw, B.D3TOM_LINEAR_RESIDUAL, out, tile, residual=tr)
    torch.cuda.synchronize()
    _one_step(_host(out), OS.round_bf16(r.astype(np.float64) + ref), "residual")
    # in place on the residual buffer
    B.d3tom_linear_tile(ta, tw, B.D3TOM_LINEAR_RESIDUAL, tr, tile, residual=tr)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(_host(tr), _host(out))


@pytest.mark.parametrize("M,N,K,chunk", [(77, 384, 128, 128), (493, 768, 256, 256), (10, 48, 64, 16)])
def test_linear_chunked_output(B, M, N, K, chunk):
    rng = np.random.default_rng([M, N, K, chunk])
    a = W.round_to(rng.standard_normal((M, K)).astype(np.float32), "bf16")
    w = W.round_to((rng.standard_normal((N, K)) / np.sqrt(K)).astype(np.float32), "bf16")
    ref = OS.round_bf16(OS.linear(a, w))
    out = torch.zeros(N // chunk, M, chunk, dtype=torch.bfloat16, device="cuda")
    B.d3tom_linear(_dev(a), _dev(w), B.D3TOM_LINEAR_PLAIN, out, out_chunk=chunk)
    torch.cuda.synchronize()
    got = _host(out)
    for c in range(N // chunk):
        _one_step(got[c], ref[:, c * chunk:(c + 1) * chunk], f"chunk {c}")


@pytest.mark.parametrize("tile", [1, 2, 4])
@pytest.mark.parametrize("M,F,K", [(5, 64, 64), (200, 96, 128), (493, 704, 256), (130, 1408, 512)])
def test_linear_swiglu(B, M, F, K, tile):
    rng = np.random.default_rng([M, F, K])
    a = W.round_to(rng.standard_normal((M, K)).astype(np.float32), "bf16")
    w = W.round_to((2.0 * rng.standard_normal((2 * F, K)) / np.sqrt(K)).astype(np.float32), "bf16")
    ref = OS.round_bf16(OS.swiglu(OS.linear(a, w[:F]), OS.linear(a, w[F:])))
    out = torch.zeros(M, F, dtype=torch.bfloat16, device="cuda")
    B.d3tom_linear_tile(_dev(a), _dev(w), B.D3TOM_LINEAR_SWIGLU, out, tile)
    torch.cuda.synchronize()
    _one_step(_host(out), ref, f"swiglu {M}x{F}x{K} tile {tile}")


@pytest.mark.parametrize("height,width", [(1, 2), (1, 4), (2, 2), (2, 3), (2, 4), (4, 2), (4, 3), (4, 4)])
@pytest.mark.parametrize("M,N,K", [(1, 8, 64), (257, 392, 192), (300, 520, 576)])       # one row; one past a tile, odd ring tails
def test_linear_every_tile(B, M, N, K, height, width):
    rng = np.random.default_rng([M, N, K, width])
    a = W.round_to(rng.standard_normal((M, K)).astype(np.float32), "bf16")
    w = W.round_to((2.0 * rng.standard_normal((2 * N, K)) / np.sqrt(K)).astype(np.float32), "bf16")
    r = W.round_to(rng.standard_normal((M, N)).astype(np.float32), "bf16")
    ta, tw, tr = _dev(a), _dev(w), _dev(r)
    out = torch.full((M, N), 7.0, dtype=torch.bfloat16, device="cuda")
    B.d3tom_linear_tile(ta, tw[:N].contiguous(), B.D3TOM_LINEAR_RESIDUAL, out, height + 16 * width, residual=tr)
    act = torch.full((M, N), 7.0, dtype=torch.bfloat16, device="cuda")
    B.d3tom_linear_tile(ta, tw, B.D3TOM_LINEAR_SWIGLU, act, height + 16 * width)
    torch.cuda.synchronize()
    up = OS.linear(a, w[N:])
    _one_step(_host(out), OS.round_bf16(r.astype(np.float64) + OS.linear(a, w[:N])), "residual")
    _one_step(_host(act), OS.round_bf16(OS.swiglu(OS.linear(a, w[:N]), up)), "swiglu")


# what the estimate never takes with the stack's epilogues
NOT_BUILT = [("slices", t) for t in ("64x256", "128x192 loaders", "128x256", "160x256", "192x256", "224x256", "256x128 loaders", "256x192", "256x256")]
NOT_BUILT += [("rope", "64x256"), ("rope", "256x128")]


@pytest.mark.parametrize("stages,rows_over,cols_over", [(1, 1, -8), (3, -3, 40), (7, 0, 8), (12, 1, 72)])     # ring tails; remainders of a tile
@pytest.mark.parametrize("epilogue", ["plain", "residual", "swiglu", "slices", "rope"])
@pytest.mark.parametrize("index", range(len(LIN_TILES)))
def test_linear_every_tile_with_every_epilogue(B, index, epilogue, stages, rows_over, cols_over):
    """Operands of -1, 0 and 1: every product is a whole number below 256, so the sums are exact in float32 and in bf16."""
    bm, bn = (int(x) for x in LIN_TILES[index].split()[0].split("x"))
    M, N, K = 2 * bm + rows_over, 3 * bn + cols_over, 64 * stages
    rng = np.random.default_rng([index, stages])
    ints = lambda *sh: rng.integers(-1, 2, sh).astype(np.float32)
    a, w = ints(M, K), ints(2 * N, K)
    full = a.astype(np.float64) @ w.T.astype(np.float64)
    prod = full[:, :N]
    assert np.abs(full).max() <= 256
    ta, tw = _dev(a), _dev(w[:N])
    out = torch.full((M, N), 7.0, dtype=torch.bfloat16, device="cuda")
    if (epilogue, LIN_TILES[index]) in NOT_BUILT:
        with pytest.raises(B.D3tomError) as e:
            if epilogue == "slices":
                B.d3tom_linear_pinned(ta, tw, B.D3TOM_LINEAR_PARTIAL, torch.empty(M, N, device="cuda"), index)
            else:
                B.d3tom_linear_pinned(ta, _dev(w[:192]), B.D3TOM_LINEAR_ROPE, out, index, extra=torch.empty(M, 64, device="cuda"), out_chunk=64, rope_dh=64)
        assert e.value.status == B.D3TOM_ERR_UNSUPPORTED
        return
    if epilogue == "plain":
        B.d3tom_linear_pinned(ta, tw, B.D3TOM_LINEAR_PLAIN, out, index)
        np.testing.assert_array_equal(_host(out), prod)
        ch = torch.full((N // 8, M, 8), 7.0, dtype=torch.bfloat16, device="cuda")
        B.d3tom_linear_pinned(ta, tw, B.D3TOM_LINEAR_PLAIN, ch, index, out_chunk=8)
        np.testing.assert_array_equal(_host(ch).transpose(1, 0, 2).reshape(M, N), prod)
    elif epilogue == "residual":
        r = rng.integers(-100, 101, (M, N)).astype(np.float32)
        B.d3tom_linear_pinned(ta, tw, B.D3TOM_LINEAR_RESIDUAL, out, index, extra=_dev(r))
        np.testing.assert_array_equal(_host(out), OS.round_bf16(prod + r))
    elif epilogue == "swiglu":
        B.d3tom_linear_pinned(ta, _dev(w), B.D3TOM_LINEAR_SWIGLU, out, index)
        _one_step(_host(out), OS.round_bf16(OS.swiglu(prod, full[:, N:])), "swiglu")
    elif epilogue == "slices":
        for slices in (1, 2, 4):
            ak, wk = ints(M, K * slices), ints(N, K * slices)
            part = torch.full((slices, M, N), 7.0, device="cuda")
            B.d3tom_linear_pinned(_dev(ak), _dev(wk), B.D3TOM_LINEAR_PARTIAL, part, index, slices=slices)
            for i in range(slices):
                np.testing.assert_array_equal(part[i].cpu().numpy(), ak[:, i * K:(i + 1) * K] @ wk[:, i * K:(i + 1) * K].T)
    else:
        for dh, d in ((64, 192), (128, 384)):
            wq = ints(3 * d, K)
            ang = rng.uniform(-200, 200, (M, dh // 2))
            cs = np.stack([np.cos(ang), np.sin(ang)], axis=2).astype(np.float32)
            qkv = torch.full((3, M, d), 7.0, dtype=torch.bfloat16, device="cuda")
            B.d3tom_linear_pinned(ta, _dev(wq), B.D3TOM_LINEAR_ROPE, qkv, index, extra=torch.from_numpy(cs).cuda(), out_chunk=d, rope_dh=dh)
            ref = (a.astype(np.float64) @ wq.T).reshape(M, 3, d // dh, 2, dh // 2)
            x0, x1, c, sn = ref[:, :2, :, 0], ref[:, :2, :, 1], cs[:, None, None, :, 0].astype(np.float64), cs[:, None, None, :, 1].astype(np.float64)
            ref[:, :2, :, 0], ref[:, :2, :, 1] = x0 * c - x1 * sn, x1 * c + x0 * sn
            ref = ref.transpose(1, 0, 2, 3, 4).reshape(3, M, d)
            np.testing.assert_array_equal(_host(qkv)[2], ref[2])
            _one_step(_host(qkv)[:2], OS.round_bf16(ref[:2]), "rope")


# (rows, rows of w, contraction) for which the library takes the tile named, ragged in both directions; the last is cut into two launches
LIN_CHOSEN = [("64x64 loaders", 100, 1008, 64), ("64x64 loaders", 100, 48, 64), ("64x96 loaders", 70, 12288, 4096), ("64x96 loaders", 250, 4112, 64), ("64x128 loaders", 1500, 1008, 64),
              ("96x128 loaders", 900, 3008, 64), ("128x128", 700, 4112, 2048), ("128x192 loaders", 500, 12288, 320), ("128x256", 300, 16400, 640),
              ("160x128 loaders", 1500, 3008, 320), ("160x128 loaders", 3300, 3008, 320), ("160x256", 300, 22016, 1024),
              ("192x128 loaders", 1300, 4112, 640), ("192x128 loaders", 2500, 4112, 320), ("192x256", 493, 16400, 1024), ("224x256", 3000, 4112, 1024),
              ("256x128 loaders", 1850, 4080, 4096), ("256x128 loaders", 2050, 3008, 320), ("256x128 loaders", 3000, 4112, 320),
              ("256x192", 493, 22016, 2048), ("256x256", 700, 16400, 2048), ("256x256 + 64x64 loaders", 1400, 22016, 4096)]


@pytest.mark.parametrize("tile,M,N,K", LIN_CHOSEN)
def test_linear_chosen_tiles(B, tile, M, N, K):
    """Every tile the estimate can choose, with both kinds of epilogue, against float32 products of the same bf16 values."""
    assert _chosen(M, N, K) == tile
    g = torch.Generator(device="cuda"); g.manual_seed(M + N)
    rnd = lambda *sh: torch.randn(*sh, generator=g, device="cuda")
    a, w, r = rnd(M, K).bfloat16(), (2.0 * rnd(N, K) / np.sqrt(K)).bfloat16(), rnd(M, N).bfloat16()
    prod = a.float() @ w.float().t()
    out = torch.full((M, N), 7.0, dtype=torch.bfloat16, device="cuda")
    act = torch.full((M, N // 2), 7.0, dtype=torch.bfloat16, device="cuda")
    B.d3tom_linear(a, w, B.D3TOM_LINEAR_RESIDUAL, out, residual=r)
    B.d3tom_linear(a, w, B.D3TOM_LINEAR_SWIGLU, act)
    for got, ref in ((out, prod + r.float()), (act, torch.nn.functional.silu(prod[:, :N // 2]) * prod[:, N // 2:])):
        # one bf16 step and the two sides' float32 sums, as in _one_step
        excess = ((got.float() - ref).abs() - 2.0 ** -7 * ref.abs()).max().item()
        assert excess <= 1e-3 * ref.square().mean().sqrt().item(), (tile, excess)
        assert (got == ref.bfloat16()).float().mean().item() > 0.97


def test_linear_two_launch_plan(B):
    """Shapes whose tall tiles fill one round of the chip and a bit: the library cuts the columns into a
    full round of tall tiles and a remainder with smaller tiles (two launches, one result)."""
    rng = np.random.default_rng(21)
    M, K, n = 540, 2048, 22016
    assert _chosen(M, n, K) == "192x256 + 64x64 loaders"
    a = W.round_to(rng.standard_normal((M, K)).astype(np.float32), "bf16")
    w = W.round_to((rng.standard_normal((n, K)) / np.sqrt(K)).astype(np.float32), "bf16")
    r = W.round_to(rng.standard_normal((M, n)).astype(np.float32), "bf16")
    prod = OS.linear(a, w)
    ta, tw, tr = _dev(a), _dev(w), _dev(r)
    out = torch.full((M, n), 7.0, dtype=torch.bfloat16, device="cuda")
    B.d3tom_linear(ta, tw, B.D3TOM_LINEAR_RESIDUAL, out, residual=tr)
    torch.cuda.synchronize()
    _one_step(_host(out), OS.round_bf16(r.astype(np.float64) + prod), "two-launch residual")
    act = torch.full((M, n // 2), 7.0, dtype=torch.bfloat16, device="cuda")
    B.d3tom_linear(ta, tw, B.D3TOM_LINEAR_SWIGLU, act)
    torch.cuda.synchronize()
    _one_step(_host(act), OS.round_bf16(OS.swiglu(prod[:, :n // 2], prod[:, n // 2:])), "two-launch swiglu")
    ch = torch.full((n // 128, M, 128), 7.0, dtype=torch.bfloat16, device="cuda")
    B.d3tom_linear(ta, tw, B.D3TOM_LINEAR_PLAIN, ch, out_chunk=128)
    torch.cuda.synchronize()
    _one_step(_host(ch).transpose(1, 0, 2).reshape(M, n), OS.round_bf16(prod), "two-launch chunked")


def test_linear_rejects(B):
    a = torch.zeros(4, 64, dtype=torch.bfloat16, device="cuda")
    w = torch.zeros(16, 64, dtype=torch.bfloat16, device="cuda")
    out = torch.zeros(4, 16, dtype=torch.bfloat16, device="cuda")
    with pytest.raises(B.D3tomError) as e:
        B.d3tom_linear(a, w, B.D3TOM_LINEAR_RESIDUAL, out)                     # residual missing
    assert e.value.status == B.D3TOM_ERR_INVALID_ARG
    with pytest.raises(B.D3tomError) as e:
        B.d3tom_linear(a[:, :32].contiguous(), w[:, :32].contiguous(), B.D3TOM_LINEAR_PLAIN, out)   # K % 64
    assert e.value.status == B.D3TOM_ERR_UNSUPPORTED
    with pytest.raises(B.D3tomError) as e:
        B.d3tom_linear(a, w, B.D3TOM_LINEAR_PLAIN, out, out_chunk=12)
    assert e.value.status == B.D3TOM_ERR_INVALID_ARG
    with pytest.raises(B.D3tomError) as e:
        B.d3tom_linear_tile(a, w, B.D3TOM_LINEAR_PLAIN, out, 3)
    assert e.value.status == B.D3TOM_ERR_INVALID_ARG


def test_linear_full_size_samples(B):
    """The projections of the full-size stack (4096 / 11008 wide, 493 and 3773 rows) in the launch
    configuration the library picks itself; a sample of output elements against float64 dot products."""
    g = torch.Generator(device="cuda"); g.manual_seed(5)
    d, F = 4096, 11008
    for M in (493, 3773):
        a = torch.randn(M, d, generator=g, device="cuda").to(torch.bfloat16)
        for name, n_rows, K, epi in (("qkv", 3 * d, d, B.D3TOM_LINEAR_PLAIN), ("gate_up", 2 * F, d, B.D3TOM_LINEAR_SWIGLU),
                                     ("down", d, F, B.D3TOM_LINEAR_RESIDUAL)):
            w = (torch.randn(n_rows, K, generator=g, device="cuda") * 0.02).to(torch.bfloat16)
            inp = a if K == d else torch.randn(M, K, generator=g, device="cuda").to(torch.bfloat16)
            n_out = n_rows // 2 if epi == B.D3TOM_LINEAR_SWIGLU else n_rows
            res = torch.randn(M, n_out, generator=g, device="cuda").to(torch.bfloat16) if epi == B.D3TOM_LINEAR_RESIDUAL else None
            out = torch.zeros(M, n_out, dtype=torch.bfloat16, device="cuda")
            B.d3tom_linear(inp, w, epi, out, residual=res)
            torch.cuda.synchronize()
            rng = np.random.default_rng([M, n_rows])
            rows = np.unique(np.concatenate([[0, M - 1], rng.integers(0, M, 24)]))
            cols = np.unique(np.concatenate([[0, n_out - 1], rng.integers(0, n_out, 24)]))
            ah = _host(inp[torch.from_numpy(rows).cuda()])
            got = _host(out[torch.from_numpy(rows).cuda()][:, torch.from_numpy(cols).cuda()])
            if epi == B.D3TOM_LINEAR_SWIGLU:
                wg = _host(w[torch.from_numpy(cols).cuda()]); wu = _host(w[torch.from_numpy(cols + n_out).cuda()])
                ref = OS.swiglu(OS.linear(ah, wg), OS.linear(ah, wu))
            else:
                ref = OS.linear(ah, _host(w[torch.from_numpy(cols).cuda()]))
                if res is not None:
                    ref = ref + _host(res[torch.from_numpy(rows).cuda()][:, torch.from_numpy(cols).cuda()])
            _one_step(got, OS.round_bf16(ref), f"{name} M={M}")
            del w, out


# ---- the whole step ----------------------------------------------------------------------------
def _gpu_blocks(case):
    blocks = []
    for b in case["blocks"]:
        blocks.append(dict(attn_norm=_dev(b["attn_norm"]), w_qkv=_dev(np.concatenate([b["wq"], b["wk"], b["wv"]], axis=0)),
                           w_o=_dev(b["wo"]), ffn_norm=_dev(b["ffn_norm"]),
                           w_gate_up=_dev(np.concatenate([b["w_gate"], b["w_up"]], axis=0)), w_down=_dev(b["w_down"])))
    return blocks


def _run_stack(B, case, keep_k, merge_layer, D=None, mode=0, eps=1e-5, theta=10000.0):
    N, d, H, F, L, V = case["N"], case["d"], case["H"], case["F"], case["L"], case["V"]
    D = case["D"] if D is None else D
    gb = _gpu_blocks(case)
    arr = B.block_weights(gb)
    ws = B.workspace(B.d3tom_stack_workspace_bytes(N, d, H, F, V, max(D, 1)))
    y = torch.zeros(N, d, dtype=torch.bfloat16, device="cuda")
    src = torch.full((N,), -1, dtype=torch.int32, device="cuda")
    scores = torch.zeros(V, dtype=torch.float32, device="cuda")
    kept = torch.zeros(max(keep_k, 1), dtype=torch.int32, device="cuda")
    asg = torch.zeros(V, dtype=torch.int32, device="cuda")
    dec = torch.from_numpy(case["dec_idx"][:D].copy()).cuda() if D > 0 else None
    x = _dev(case["x"])
    n_out = B.d3tom_stack_step(x, H, F, arr, L, merge_layer, dec, D, case["vis_start"], V, keep_k, mode, eps, theta, y, ws,
                               src_pos=src, scores=scores, kept_idx=kept, assign=asg)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(_host(x), case["x"].astype(np.float64))       # the input is never written
    return dict(n_out=n_out, y=_host(y[:n_out]), src_pos=src[:n_out].cpu().numpy(), S=scores.cpu().numpy(),
                kept=kept.cpu().numpy(), assign=asg.cpu().numpy())


def _oracle_blocks(case):
    return [OS.Block(**b) for b in case["blocks"]]


STACK_CASES = [
    # L, d, H, F, P, V, O, D, keep_k, merge_layer
    (4, 256, 4, 512, 32, 144, 32, 16, 36, 2),          # the tiny configuration's sequence, four blocks
    (3, 512, 4, 704, 20, 729, 40, 9, 100, 1),          # one crop of visual tokens, head size 128, merge in block 1
    (3, 256, 2, 320, 7, 300, 21, 5, 299, 3),           # merge in the last block, one token merged away
    (2, 256, 4, 512, 0, 200, 8, 8, 1, 1),              # no prompt, everything merged into one token
    (2, 2048, 16, 2048, 10, 120, 20, 6, 30, 1),        # wide enough that the output / down projections are split along k
    (2, 192, 3, 320, 5, 90, 11, 4, 30, 1),             # three heads of 64: a 128-column projection tile straddles q | k and k | v
]


def _merge_block_inputs(B, case, l_star, eps=1e-5, theta=10000.0):
    """What the merge layer of block l_star sees on the GPU: the block's rotated q, k and its post-attention
    hidden state, rebuilt from the same entry points in the same order (the kernels are deterministic, so
    these are the very values inside d3tom_stack_step, up to the order of the float32 sums of an output projection
    that the step cuts along its contraction, and of the attention above 512 tokens, where the step does without the 64-query tiles that
    d3tom_attend takes for few heads)."""
    N, d, H, F, V = case["N"], case["d"], case["H"], case["F"], case["V"]
    dh = d // H
    x = _dev(case["x"])
    if l_star > 1:
        sub = dict(case, L=l_star - 1, blocks=case["blocks"][:l_star - 1])
        h = _dev(_run_stack(B, sub, 1, 0, D=0)["y"])
    else:
        h = x
    blk = _gpu_blocks(dict(blocks=[case["blocks"][l_star - 1]]))[0]
    a = torch.empty_like(h)
    B.d3tom_rmsnorm(h, blk["attn_norm"], eps, a)
    qkv = torch.empty(3, N, d, dtype=torch.bfloat16, device="cuda")
    B.d3tom_linear(a, blk["w_qkv"], B.D3TOM_LINEAR_PLAIN, qkv, out_chunk=d)
    q, k, v = (qkv[i].view(N, H, dh) for i in range(3))
    pos = torch.arange(N, dtype=torch.int32, device="cuda")
    B.d3tom_rope(q, k, pos, theta)
    o = torch.empty(N, H, dh, dtype=torch.bfloat16, device="cuda")
    cu = torch.tensor([0, N], dtype=torch.int32, device="cuda")
    B.d3tom_attend(q, k, v, cu, N, 1.0 / np.sqrt(dh), o, B.workspace(256))
    ht = torch.empty(N, d, dtype=torch.bfloat16, device="cuda")
    B.d3tom_linear(o.view(N, d), blk["w_o"], B.D3TOM_LINEAR_RESIDUAL, ht, residual=h)
    torch.cuda.synchronize()
    return _host(q).astype(np.float32), _host(k).astype(np.float32), _host(ht).astype(np.float32)


@pytest.mark.parametrize("L,d,H,F,Pn,V,O,D,keep_k,l_star", STACK_CASES)
def test_stack_step_against_oracle(B, L, d, H, F, Pn, V, O, D, keep_k, l_star):
    case = W.stack_case(L * 1000 + V, L=L, d=d, H=H, F=F, P=Pn, V=V, O=O, D=D, std=1.0 / np.sqrt(d), gain_jitter=0.1)
    got = _run_stack(B, case, keep_k, l_star)
    assert got["n_out"] == case["N"] - (V - keep_k)
    # 1. the merge layer inside the stack, stage by stage, on the values the GPU itself fed to it
    q, k, ht = _merge_block_inputs(B, case, l_star)
    S_ref = oracle.importance(q, k, case["dec_idx"], case["vis_start"], V)
    P.check_scores(got["S"], S_ref)
    slot = np.full(V, -1, np.int32); slot[got["kept"]] = np.arange(keep_k)
    P.check_kept(got["kept"], slot, S_ref, keep_k)
    P.check_assign(got["assign"], ht, case["vis_start"], V, got["kept"])
    # 2. the whole step against the oracle's whole step.  The oracle's own hidden states differ from the
    # GPU's by single bf16 steps here and there, which moves its scores by up to ~1e-2 relative, so its own
    # top-k may differ near the threshold: it is told the GPU's (checked) kept set and assignment.
    ref = stack_step_given(case["x"], _oracle_blocks(case), H, case["dec_idx"], case["vis_start"], V, keep_k, l_star,
                           kept=got["kept"], assign=got["assign"])
    np.testing.assert_array_equal(got["src_pos"], ref["src_pos"])
    # Tolerance: a float32 pipeline differs from the float64 one by a few float32 ulps in every value it is
    # about to store; where that crosses a bf16 rounding boundary the stored value moves by one bf16 step,
    # and later blocks carry such steps on.  The oracle measures that floor on itself (same step, every
    # stored value perturbed by 3e-7 relative before rounding); the GPU must stay within 3x of it.
    alt = stack_step_given(case["x"], _oracle_blocks(case), H, case["dec_idx"], case["vis_start"], V, keep_k, l_star,
                           kept=got["kept"], assign=got["assign"], store=jittered_bf16(3e-7, 1))
    rms = lambda a, b: np.sqrt(np.mean((a - b) ** 2)) / np.sqrt(np.mean(b ** 2))
    y, yr = got["y"], ref["y"]
    floor, rel = rms(alt["y"], yr), rms(y, yr)
    floor_s = (np.abs(alt["S"] - ref["S"]) / np.abs(ref["S"])).max()
    rel_s = (np.abs(got["S"] - ref["S"]) / np.abs(ref["S"])).max()
    print(f"stack L={L} d={d}: rel rms {rel:.2e} (floor {floor:.2e}), max abs {np.abs(y - yr).max():.2e} "
          f"(floor {np.abs(alt['y'] - yr).max():.2e}), score rel {rel_s:.2e} (floor {floor_s:.2e})")
    assert rel <= 3.0 * floor + 1e-4, (rel, floor)
    assert np.abs(y - yr).max() <= 3.0 * np.abs(alt["y"] - yr).max() + 2.0 ** -8, np.abs(y - yr).max()
    assert (np.abs(y - yr) - _whole_step_elementwise_bound(yr, L)).max() <= 0
    assert rel_s <= 3.0 * floor_s + 1e-3, (rel_s, floor_s)


def test_stack_step_without_deciders_runs_full_length(B):
    case = W.stack_case(77, L=3, d=256, H=4, F=512, P=16, V=100, O=12, D=4, std=1.0 / 16, gain_jitter=0.1)
    got = _run_stack(B, case, 10, 2, D=0)
    assert got["n_out"] == case["N"]
    np.testing.assert_array_equal(got["src_pos"], np.arange(case["N"]))
    ref = OS.stack_step(case["x"], _oracle_blocks(case), case["H"], None, case["vis_start"], case["V"], 10, 2)
    alt = OS.stack_step(case["x"], _oracle_blocks(case), case["H"], None, case["vis_start"], case["V"], 10, 2,
                        store=jittered_bf16(3e-7))
    rms = lambda a, b: np.sqrt(np.mean((a - b) ** 2)) / np.sqrt(np.mean(b ** 2))
    assert rms(got["y"], ref["y"]) <= 3.0 * rms(alt["y"], ref["y"]) + 1e-4
    # keeping every visual token is the same computation: the merge copies rows bit-exactly
    keep_all = _run_stack(B, case, case["V"], 2)
    np.testing.assert_array_equal(keep_all["y"], got["y"])
    np.testing.assert_array_equal(keep_all["src_pos"], got["src_pos"])
    # a merge layer outside 1 .. L never merges
    off = _run_stack(B, case, 10, 0)
    np.testing.assert_array_equal(off["y"], got["y"])


@pytest.mark.parametrize("V", [450, 520, 1300])
def test_spellings_of_the_unmerged_model_agree(B, V):
    """No deciders, a merge layer outside 1 .. L and every token kept are one model, bit for bit, on both sides of the length up to
    which attention runs on its short-sample kernel (512 tokens)."""
    case = W.stack_case(81, L=2, d=256, H=2, F=320, P=8, V=V, O=12, D=3, std=1.0 / 16, gain_jitter=0.1)
    plain = _run_stack(B, case, 10, 0, D=0)
    for got in (_run_stack(B, case, 10, 2, D=0), _run_stack(B, case, 10, 1, D=0), _run_stack(B, case, 10, 0), _run_stack(B, case, V, 1)):
        np.testing.assert_array_equal(got["y"], plain["y"])


@pytest.mark.parametrize("n,others", [(600, [520, 777, 600] * 5), (530, [1500]), (700, [3, 40, 513])])
def test_rows_of_a_sample_do_not_depend_on_its_companions(B, n, others):
    """Above 512 tokens the unmerged blocks of a stack give a sample the same bits alone (few tiles of queries) and in a batch (more and wider
    ones): what a merge decides near-ties by does not move with the number of samples."""
    d, H, F = 256, 4, 320
    case = W.stack_case(84, L=2, d=d, H=H, F=F, P=8, V=n - 20, O=12, D=3, std=1.0 / 16, gain_jitter=0.1)
    gb = _gpu_blocks(case)
    arr = B.block_weights(gb)
    x = _dev(case["x"])
    outs = []
    for rest in ([], others):
        N = rest + [n]
        rows = torch.cat([torch.randn(sum(rest), d, device="cuda").to(torch.bfloat16), x])
        y = torch.zeros_like(rows)
        ws = B.workspace(B.d3tom_stack_batch_workspace_bytes(len(N), sum(N), max(N), d, H, F, 0, 0, 1))
        z = [0] * len(N)
        B.d3tom_stack_step_batch(rows, N, H, F, arr, 2, 0, None, z, z, z, z, 0, 1e-5, 10000.0, y, ws)
        torch.cuda.synchronize()
        outs.append(y[-n:].clone())
    assert torch.equal(*outs)


def test_stack_step_sum_mode(B):
    case = W.stack_case(78, L=2, d=256, H=4, F=512, P=8, V=120, O=12, D=6, std=1.0 / 16, gain_jitter=0.1)
    got = _run_stack(B, case, 30, 1, mode=1)
    ref = stack_step_given(case["x"], _oracle_blocks(case), case["H"], case["dec_idx"], case["vis_start"], case["V"], 30, 1,
                           kept=got["kept"], assign=got["assign"], mode="sum")
    alt = stack_step_given(case["x"], _oracle_blocks(case), case["H"], case["dec_idx"], case["vis_start"], case["V"], 30, 1,
                           kept=got["kept"], assign=got["assign"], mode="sum", store=jittered_bf16(3e-7))
    rms = lambda a, b: np.sqrt(np.mean((a - b) ** 2)) / np.sqrt(np.mean(b ** 2))
    assert rms(got["y"], ref["y"]) <= 3.0 * rms(alt["y"], ref["y"]) + 1e-4


def test_stack_step_rejects(B):
    case = W.stack_case(79, L=1, d=256, H=4, F=512, P=4, V=40, O=4, D=2, std=1.0 / 16)
    gb = _gpu_blocks(case)
    arr = B.block_weights(gb)
    x = _dev(case["x"])
    y = torch.zeros_like(x)
    ws = B.workspace(B.d3tom_stack_workspace_bytes(case["N"], 256, 4, 512, 40, 2))
    dec = torch.from_numpy(case["dec_idx"]).cuda()
    args = dict(mode=0, eps=1e-5, theta=10000.0, y=y, ws=ws)
    with pytest.raises(B.D3tomError) as e:       # kept count outside 1 .. V
        B.d3tom_stack_step(x, 4, 512, arr, 1, 1, dec, 2, 4, 40, 41, **args)
    assert e.value.status == B.D3TOM_ERR_INVALID_ARG
    with pytest.raises(B.D3tomError) as e:       # head size the attention kernel is not built for
        B.d3tom_stack_step(x, 8, 512, arr, 1, 1, dec, 2, 4, 40, 10, **args)
    assert e.value.status == B.D3TOM_ERR_UNSUPPORTED
    with pytest.raises(B.D3tomError) as e:
        B.d3tom_stack_step(x, 4, 512, arr, 1, 1, dec, 2, 4, 40, 10, mode=0, eps=1e-5, theta=10000.0, y=y, ws=ws[:1024])
    assert e.value.status == B.D3TOM_ERR_WORKSPACE_TOO_SMALL
    for theta in (1.0, 0.5, 0.0, -1.0, float("nan"), float("inf"), 3.2e38):
        bad = dict(args, theta=theta)
        for D in (2, 0):
            with pytest.raises(B.D3tomError) as e:
                B.d3tom_stack_step(x, 4, 512, arr, 1, 1, dec, D, 4, 40, 10, **bad)
            assert e.value.status == B.D3TOM_ERR_INVALID_ARG
            with pytest.raises(B.D3tomError) as e:
                B.d3tom_stack_step_batch(x, [case["N"]], 4, 512, arr, 1, 1, dec, [D], [4], [40], [10], **bad)
            assert e.value.status == B.D3TOM_ERR_INVALID_ARG


@pytest.mark.parametrize("merging", [True, False])
@pytest.mark.parametrize("merge_layer", [1, 2, 3])
def test_stack_step_optional_outputs_are_only_written(B, merge_layer, merging):
    """A caller who has no use for the optional outputs may pass one array for all of them: they spoil each other and nothing else."""
    case = W.stack_case(83, L=3, d=256, H=4, F=512, P=6, V=300, O=9, D=4, std=1.0 / 16, gain_jitter=0.1)
    gb = _gpu_blocks(case)
    x, arr = _dev(case["x"]), B.block_weights(gb)
    dec = torch.from_numpy(case["dec_idx"]).cuda() if merging else None
    ws = B.workspace(B.d3tom_stack_workspace_bytes(case["N"], 256, 4, 512, 300, 4))
    dummy = torch.zeros(case["N"], dtype=torch.int32, device="cuda")
    ys = []
    for extra in (dict(), dict(src_pos=dummy, scores=dummy.view(torch.float32), kept_idx=dummy, assign=dummy)):
        y = torch.zeros_like(x)
        n = B.d3tom_stack_step(x, 4, 512, arr, 3, merge_layer, dec, 4 if merging else 0, 6, 300, 120, 0, 1e-5, 10000.0, y, ws, **extra)
        torch.cuda.synchronize()
        ys.append(y[:n].clone())
    assert torch.equal(*ys)


# ---- full-size shapes (hidden 4096, 32 x 128 heads, SwiGLU 11008, 3645 + 64 + 64 tokens) --------------------
def _full_size(B, L):
    cfg = dict(W.STACK_3645, L=L)
    inp = W.stack_device_inputs(cfg)
    N = cfg["P"] + cfg["V"] + cfg["O"]
    ws = B.workspace(B.d3tom_stack_workspace_bytes(N, cfg["d"], cfg["H"], cfg["F"], cfg["V"], 64))
    return cfg, inp, N, ws


def _step_full(B, cfg, inp, N, ws, L, merge_layer, D, keep_k, want=()):
    y = torch.zeros(N, cfg["d"], dtype=torch.bfloat16, device="cuda")
    src = torch.full((N,), -1, dtype=torch.int32, device="cuda")
    extra = dict(scores=torch.zeros(cfg["V"], dtype=torch.float32, device="cuda"),
                 kept_idx=torch.zeros(cfg["V"], dtype=torch.int32, device="cuda"),
                 assign=torch.zeros(cfg["V"], dtype=torch.int32, device="cuda"))
    dec = (cfg["P"] + cfg["V"] + torch.arange(0, 2 * D, 2, dtype=torch.int32, device="cuda")) if D else None
    arr = B.block_weights(inp["blocks"][:L])
    n_out = B.d3tom_stack_step(inp["x"], cfg["H"], cfg["F"], arr, L, merge_layer, dec, D, cfg["P"], cfg["V"], keep_k, 0,
                               cfg["eps"], cfg["theta"], y, ws, src_pos=src, **extra)
    torch.cuda.synchronize()
    return dict(n_out=n_out, y=y[:n_out], src_pos=src[:n_out].cpu().numpy(), S=extra["scores"].cpu().numpy(),
                kept=extra["kept_idx"][:keep_k].cpu().numpy(), assign=extra["assign"].cpu().numpy(),
                dec=dec.cpu().numpy() if D else None)


def test_stack_full_size_properties(B):
    """Properties that hold at any size, on the full-size shapes in the launch configuration the benchmark
    times (merge inside block 3): keeping every token or having no deciders is the unmerged model, bit for
    bit; a merged step returns the kept tokens in place, at their original positions."""
    cfg, inp, N, ws = _full_size(B, 4)
    P_, V = cfg["P"], cfg["V"]
    k = B.d3tom_keep_count(V, cfg["keep_ratio"])
    plain = _step_full(B, cfg, inp, N, ws, 4, 3, 0, k)
    assert plain["n_out"] == N and bool(torch.isfinite(plain["y"].float()).all())
    keep_all = _step_full(B, cfg, inp, N, ws, 4, 3, 8, V)
    assert torch.equal(keep_all["y"], plain["y"])
    np.testing.assert_array_equal(keep_all["src_pos"], np.arange(N))
    merged = _step_full(B, cfg, inp, N, ws, 4, 3, 8, k)
    assert merged["n_out"] == N - (V - k) == 493 and bool(torch.isfinite(merged["y"].float()).all())
    kept = merged["kept"]
    assert np.all(np.diff(kept) > 0) and kept.min() >= 0 and kept.max() < V
    np.testing.assert_array_equal(merged["src_pos"], np.concatenate([np.arange(P_), P_ + kept, np.arange(P_ + V, N)]))
    # the kept tokens are the k best scores
    S = merged["S"]
    assert S[kept].min() >= np.delete(S, kept).max()
    np.testing.assert_array_equal(merged["assign"][kept], np.arange(k))
    # the same step twice gives the same bits (no float atomics anywhere on the path)
    again = _step_full(B, cfg, inp, N, ws, 4, 3, 8, k)
    assert torch.equal(again["y"], merged["y"])


def _whole_step_elementwise_bound(ref, n_blocks):
    """Element-wise bound of a whole step.  The last rounding of an element can differ by one bf16 step:
    2^-7 |ref|.  Everything before it reaches the element through normalisations and matrix products, which
    spread the rounding differences of earlier stored tensors over all elements of a row: a stored tensor
    carries a relative rms rounding error of 2^-9 / sqrt(3), a step crosses about ten stored tensors per block
    (normalised rows, q, k, v, attention output, post-attention state, merged rows, normalised rows, activation,
    block output), and independent errors add in quadrature: sigma = 2^-9 / sqrt(3) * sqrt(10 L) relative to the
    rms of the output (5e-3 for two blocks, which is the floor the oracle measures on itself).  An element's
    share of that is close to Gaussian; 8 sigma covers the largest of a few million elements."""
    rms = np.sqrt(np.mean(ref * ref)) + 1e-30
    sigma = 2.0 ** -9 / np.sqrt(3.0) * np.sqrt(10.0 * n_blocks)
    return 2.0 ** -7 * np.abs(ref) + 8.0 * sigma * rms


def test_stack_full_size_two_blocks_against_oracle(B):
    """Two full-size blocks with the merge inside the first (3773 -> 493 tokens) against the oracle: the merge
    layer stage by stage on the values the GPU itself fed to it (rebuilt through the same entry points), at the
    bars of the hot path (scores 1e-3 relative, kept set and assignment exact up to 1e-3 near-ties, every row
    checked); then the whole step, element by element and in relative rms."""
    cfg, inp, N, ws = _full_size(B, 2)
    H, V, P_ = cfg["H"], cfg["V"], cfg["P"]
    d, F, dh = cfg["d"], cfg["F"], cfg["d"] // cfg["H"]
    k = B.d3tom_keep_count(V, cfg["keep_ratio"])
    got = _step_full(B, cfg, inp, N, ws, 2, 1, 8, k)
    # 1. what the merge layer of block 1 saw on the GPU: rotated q, k and the post-attention hidden state
    blk = inp["blocks"][0]
    x_dev = inp["x"]
    a = torch.empty_like(x_dev)
    B.d3tom_rmsnorm(x_dev, blk["attn_norm"], cfg["eps"], a)
    qkv = torch.empty(3, N, d, dtype=torch.bfloat16, device="cuda")
    B.d3tom_linear(a, blk["w_qkv"], B.D3TOM_LINEAR_PLAIN, qkv, out_chunk=d)
    qd, kd, vd = (qkv[i].view(N, H, dh) for i in range(3))
    B.d3tom_rope(qd, kd, torch.arange(N, dtype=torch.int32, device="cuda"), cfg["theta"])
    o = torch.empty(N, H, dh, dtype=torch.bfloat16, device="cuda")
    B.d3tom_attend(qd, kd, vd, torch.tensor([0, N], dtype=torch.int32, device="cuda"), N, 1.0 / np.sqrt(dh), o, B.workspace(256))
    ht = torch.empty(N, d, dtype=torch.bfloat16, device="cuda")
    B.d3tom_linear(o.view(N, d), blk["w_o"], B.D3TOM_LINEAR_RESIDUAL, ht, residual=x_dev)
    torch.cuda.synchronize()
    qh, kh, hth = (t.float().cpu().numpy() for t in (qd, kd, ht))
    S_ref = oracle.importance(qh, kh, got["dec"], P_, V)
    rel_s = P.check_scores(got["S"], S_ref)
    slot = np.full(V, -1, np.int32); slot[got["kept"]] = np.arange(k)
    n_kept = P.check_kept(got["kept"], slot, S_ref, k)
    n_asg = P.check_assign(got["assign"], hth, P_, V, got["kept"])          # every pruned row
    # 2. the whole step against the oracle's whole step on the GPU's (checked) kept set and assignment
    blocks = []
    for b in inp["blocks"][:2]:
        wqkv = b["w_qkv"].float().cpu().numpy(); wgu = b["w_gate_up"].float().cpu().numpy()
        blocks.append(OS.Block(b["attn_norm"].float().cpu().numpy(), wqkv[:d], wqkv[d:2 * d], wqkv[2 * d:],
                               b["w_o"].float().cpu().numpy(), b["ffn_norm"].float().cpu().numpy(), wgu[:F], wgu[F:],
                               b["w_down"].float().cpu().numpy()))
    x = inp["x"].float().cpu().numpy()
    kw = dict(kept=got["kept"], assign=got["assign"], eps=cfg["eps"], theta=cfg["theta"])
    ref = stack_step_given(x, blocks, H, got["dec"], P_, V, k, 1, **kw)
    alt = stack_step_given(x, blocks, H, got["dec"], P_, V, k, 1, store=jittered_bf16(3e-7, 1), **kw)
    np.testing.assert_array_equal(got["src_pos"], ref["src_pos"])
    y = got["y"].float().cpu().numpy().astype(np.float64)
    rms = lambda a_, b_: np.sqrt(np.mean((a_ - b_) ** 2)) / np.sqrt(np.mean(b_ ** 2))
    rel, floor = rms(y, ref["y"]), rms(alt["y"], ref["y"])
    err, err_floor = np.abs(y - ref["y"]), np.abs(alt["y"] - ref["y"])
    print(f"full-size two blocks: rel rms {rel:.2e} (floor {floor:.2e}), max abs {err.max():.2e} (floor {err_floor.max():.2e}), "
          f"score rel {rel_s:.2e}, kept excused {n_kept}, assign excused {n_asg}")
    assert rel <= 3.0 * floor + 1e-4, (rel, floor)                         # at the rounding floor the oracle measures on itself
    assert err.max() <= 3.0 * err_floor.max() + 2.0 ** -8, (err.max(), err_floor.max())
    excess = err - _whole_step_elementwise_bound(ref["y"], 2)
    assert excess.max() <= 0, f"element-wise bound exceeded by {excess.max():.3e}"


def test_stack_trajectory_with_decider_updates(B):
    """A whole denoising trajectory (T = 9 steps) of a small stack the way the benchmark drives the full one:
    decider set from two successive token-id states on the device, embedding of the current response tokens, one
    stack step.  Step 0 has no deciders and runs unmerged (Algorithm 1); every later step merges, with a decider
    set that changes from step to step (one to several newly revealed positions)."""
    L, d, H, F, Pn, V, O, keep_k = 2, 256, 4, 512, 6, 80, 18, 20
    T = 9
    case = W.stack_case(91, L=L, d=d, H=H, F=F, P=Pn, V=V, O=O, D=0, std=1.0 / 16, gain_jitter=0.1)
    N = case["N"]
    mask_id = 126336
    states = W.mask_trajectory(5, Pn + V, O, T, mask_id)
    rng = np.random.default_rng(17)
    table = W.round_to(rng.standard_normal((64, d)).astype(np.float32), "bf16")
    mask_vec = W.round_to(rng.standard_normal(d).astype(np.float32), "bf16")
    gb = _gpu_blocks(case)
    arr = B.block_weights(gb)
    ws = B.workspace(B.d3tom_stack_workspace_bytes(N, d, H, F, V, 16))
    seq_off = torch.tensor([0, N], dtype=torch.int32, device="cuda")
    dec_idx = torch.zeros(16, dtype=torch.int32, device="cuda")
    dec_off = torch.zeros(2, dtype=torch.int32, device="cuda")
    dec_count = torch.zeros(1, dtype=torch.int32, device="cuda")
    merged_steps = 0
    sizes = set()
    for s in range(T):
        x = case["x"].copy()
        ids = states[s][Pn + V:]
        x[Pn + V:] = np.where((ids == mask_id)[:, None], mask_vec[None, :], table[ids % 64])
        D = 0
        dec_ref = np.zeros(0, np.int32)
        if s > 0:
            B.d3tom_update_deciders(torch.from_numpy(states[s - 1]).cuda(), torch.from_numpy(states[s]).cuda(), mask_id, seq_off,
                                    16, dec_idx, dec_off, dec_count)
            D = int(dec_count.item())
            dec_ref = oracle.deciders(states[s - 1], states[s], mask_id)
            np.testing.assert_array_equal(dec_idx[:D].cpu().numpy(), dec_ref)
            sizes.add(D)
        y = torch.zeros(N, d, dtype=torch.bfloat16, device="cuda")
        kept = torch.zeros(keep_k, dtype=torch.int32, device="cuda")
        asg = torch.zeros(V, dtype=torch.int32, device="cuda")
        n_out = B.d3tom_stack_step(_dev(x), H, F, arr, L, 1, dec_idx if D else None, D, Pn, V, keep_k, 0, 1e-5, 10000.0, y, ws,
                                   kept_idx=kept, assign=asg)
        torch.cuda.synchronize()
        over = dict(kept=kept.cpu().numpy(), assign=asg.cpu().numpy()) if D else {}
        ref = stack_step_given(x, _oracle_blocks(case), H, dec_ref if D else None, Pn, V, keep_k, 1, **over)
        assert n_out == ref["y"].shape[0] == (N - (V - keep_k) if D else N)
        merged_steps += int(D > 0)
        got = _host(y[:n_out])
        rel = np.sqrt(np.mean((got - ref["y"]) ** 2)) / np.sqrt(np.mean(ref["y"] ** 2))
        assert rel < 2e-2, (s, rel)          # 3x the rounding floor measured for two to four blocks
        assert (np.abs(got - ref["y"]) - _whole_step_elementwise_bound(ref["y"], L)).max() <= 0
    assert merged_steps == T - 1 and len(sizes) > 1


def test_stack_step_batch_of_ragged_samples(B):
    """Three samples of different lengths, visual blocks, decider counts and keep counts through one call: every
    sample's output against the oracle's step of that sample alone (on the kept set and assignment the GPU chose,
    which must agree with a single-sample GPU run up to near-threshold swaps); a batch that mixes samples with and
    without deciders is refused; a batch without any deciders runs unmerged."""
    L, d, H, F = 2, 256, 4, 512
    specs = [(8, 200, 12, 5, 50), (0, 96, 30, 9, 24), (20, 333, 7, 2, 111)]        # P, V, O, D, keep
    base = W.stack_case(95, L=L, d=d, H=H, F=F, P=1, V=8, O=1, D=1, std=1.0 / 16, gain_jitter=0.1)   # the shared weights
    cases = []
    for i, (Pn, V, O, D, k) in enumerate(specs):
        c = W.stack_case(96 + i, L=L, d=d, H=H, F=F, P=Pn, V=V, O=O, D=D, std=1.0 / 16, gain_jitter=0.1)
        cases.append(dict(c, blocks=base["blocks"]))
    gb = _gpu_blocks(base)
    arr = B.block_weights(gb)
    Ns = [c["N"] for c in cases]; Vs = [c["V"] for c in cases]; Ds = [c["D"] for c in cases]
    vss = [c["vis_start"] for c in cases]; ks = [sp[4] for sp in specs]
    x = _dev(np.concatenate([c["x"] for c in cases]))
    dec = torch.from_numpy(np.concatenate([c["dec_idx"] for c in cases])).cuda()
    ws = B.workspace(B.d3tom_stack_batch_workspace_bytes(3, sum(Ns), max(Ns), d, H, F, sum(Vs), max(Vs), max(Ds)))
    ws.fill_(255)
    y = torch.zeros(sum(Ns), d, dtype=torch.bfloat16, device="cuda")
    src = torch.full((sum(Ns),), -1, dtype=torch.int32, device="cuda")
    kept = torch.zeros(sum(ks), dtype=torch.int32, device="cuda")
    asg = torch.zeros(sum(Vs), dtype=torch.int32, device="cuda")
    n_out = B.d3tom_stack_step_batch(x, Ns, H, F, arr, L, 1, dec, Ds, vss, Vs, ks, 0, 1e-5, 10000.0, y, ws, src_pos=src,
                                     kept_idx=kept, assign=asg)
    torch.cuda.synchronize()
    assert n_out == [n - (v - k) for n, v, k in zip(Ns, Vs, ks)]
    yo = np.split(_host(y[:sum(n_out)]), np.cumsum(n_out)[:-1])
    so = np.split(src[:sum(n_out)].cpu().numpy(), np.cumsum(n_out)[:-1])
    ko = np.split(kept.cpu().numpy(), np.cumsum(ks)[:-1])
    ao = np.split(asg.cpu().numpy(), np.cumsum(Vs)[:-1])
    rms = lambda a_, b_: np.sqrt(np.mean((a_ - b_) ** 2)) / np.sqrt(np.mean(b_ ** 2))
    for b, c in enumerate(cases):
        ref = stack_step_given(c["x"], _oracle_blocks(c), H, c["dec_idx"], c["vis_start"], c["V"], ks[b], 1, kept=ko[b], assign=ao[b])
        alt = stack_step_given(c["x"], _oracle_blocks(c), H, c["dec_idx"], c["vis_start"], c["V"], ks[b], 1, kept=ko[b], assign=ao[b],
                               store=jittered_bf16(3e-7, 1))
        np.testing.assert_array_equal(so[b], ref["src_pos"])
        assert rms(yo[b], ref["y"]) <= 3.0 * rms(alt["y"], ref["y"]) + 1e-4
        assert (np.abs(yo[b] - ref["y"]) - _whole_step_elementwise_bound(ref["y"], L)).max() <= 0
        one = _run_stack(B, c, ks[b], 1)                       # the same sample alone through d3tom_stack_step
        assert len(np.setxor1d(one["kept"], ko[b])) <= 2
    # mixed batch: refused before anything runs; no deciders at all: every sample at full length
    with pytest.raises(B.D3tomError) as e:
        B.d3tom_stack_step_batch(x, Ns, H, F, arr, L, 1, dec, [Ds[0], 0, Ds[2]], vss, Vs, ks, 0, 1e-5, 10000.0, y, ws)
    assert e.value.status == B.D3TOM_ERR_NO_DECIDERS
    n_out = B.d3tom_stack_step_batch(x, Ns, H, F, arr, L, 1, None, [0, 0, 0], vss, Vs, ks, 0, 1e-5, 10000.0, y, ws)
    torch.cuda.synchronize()
    assert n_out == Ns
    full = np.split(_host(y), np.cumsum(Ns)[:-1])
    for b, c in enumerate(cases):
        ref = OS.stack_step(c["x"], _oracle_blocks(c), H, None, c["vis_start"], c["V"], ks[b], 1)
        alt = OS.stack_step(c["x"], _oracle_blocks(c), H, None, c["vis_start"], c["V"], ks[b], 1, store=jittered_bf16(3e-7))
        assert rms(full[b], ref["y"]) <= 3.0 * rms(alt["y"], ref["y"]) + 1e-4


def test_stack_workspace_contents_do_not_matter(B):
    case = W.stack_case(93, L=2, d=2048, H=16, F=2048, P=6, V=90, O=8, D=4, std=1.0 / 45, gain_jitter=0.1)
    N, d, H, F, V = case["N"], 2048, 16, 2048, 90
    gbs = _gpu_blocks(case)            # the pointer table below refers to these tensors: keep them alive
    arr = B.block_weights(gbs)
    x = _dev(case["x"])
    dec = torch.from_numpy(case["dec_idx"]).cuda()
    outs = []
    for fill in (0, 255):
        ws = B.workspace(B.d3tom_stack_workspace_bytes(N, d, H, F, V, 4))
        ws.fill_(fill)
        y = torch.zeros(N, d, dtype=torch.bfloat16, device="cuda")
        n_out = B.d3tom_stack_step(x, H, F, arr, 2, 1, dec, 4, case["vis_start"], V, 25, 0, 1e-5, 10000.0, y, ws)
        torch.cuda.synchronize()
        outs.append(y[:n_out].clone())
    assert torch.equal(outs[0], outs[1])
