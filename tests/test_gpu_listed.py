"""GPU parity of filtered rows that are listed (top-k / top-p leave few entries
of them) against the CPU reference, with rows of other kinds in the same
sequences: nearly flat rows (too many kept entries for a list: the sweep takes
them), rows whose largest entries lie at one end (the guess from the row's
first entries is then too high or too low), and rows that are -inf but for a
few entries. The tolerances are those of the other filter tests."""

import numpy as np
import pytest
import torch

import oracle
import paper_2505_07680_amd as sr
from workloads import level_inputs, small_shape
from workloads.gen import bf16_bits_from_f32

from gpu_util import run_accept
from test_gpu_sampling import _check_filtered, say

pytestmark = pytest.mark.gpu

# the smallest vocabularies, one granule of loads and its neighbours, odd sizes in both widths, a list's cap
VOCABS = [7, 300, 2049, 4101, 20000, 50257]


@pytest.fixture(scope="module", autouse=True)
def _library():
    sr.load()
    assert torch.cuda.is_available()
    yield
    torch.cuda.synchronize()


def _rows(z, rng):
    """Reshape the rows z [..., V] by kind, dealt over the rows in turn."""
    flat = z.reshape(-1, z.shape[-1])
    V = flat.shape[1]
    for i, row in enumerate(flat):
        kind = i % 6
        if kind == 1:  # nearly flat, on a grid so that cumulative masses move in steps
            row[:] = 0.05 * rng.integers(0, 64, V) / 64.0
        elif kind == 2:  # the largest first
            row[:] = -np.sort(-row)
        elif kind == 3:  # the largest last
            row[:] = np.sort(row)
        elif kind == 4:  # -inf but for a few
            keep = rng.permutation(V)[: min(V, 30)]
            few = row[keep].copy()
            row[:] = -np.inf
            row[keep] = few
        elif kind == 5:  # one entry far above the rest
            row[rng.integers(V)] = 40.0
    return z


def _inputs(V, logits, B, gam, seed):
    inp = level_inputs(small_shape(name=f"listed-{logits}-{V}", B=B, V=V, gamma=gam, seed=seed), kv=False)
    rng = np.random.default_rng(seed)
    p = _rows(inp.p_logits.astype(np.float32).copy(), rng)
    q = _rows(inp.q_logits.astype(np.float32).copy(), rng)
    # (a draft row related to its verifier row where the kinds agree, so that drafts are accepted too)
    G = q.shape[1]
    q[:, : G // 2] = p[:, : G // 2] + 0.25 * np.round(4 * rng.standard_normal(q[:, : G // 2].shape))
    q[np.isnan(q)] = -np.inf
    drafts = np.argmax(q + rng.gumbel(size=q.shape), axis=-1).astype(np.int32)
    if logits == "bf16":
        p, q = bf16_bits_from_f32(p), bf16_bits_from_f32(q)
    return inp, p, q, drafts


def _padded(x):
    """On the device, each sequence's rows in an allocation whose stride is a multiple of 16 bytes."""
    B, rows, V = x.shape
    x = x.view(np.int16) if x.dtype == np.uint16 else x
    per = 16 // x.itemsize
    buf = np.zeros((B, (rows * V + per - 1) // per * per), x.dtype)
    buf[:, : rows * V] = x.reshape(B, -1)
    return torch.from_numpy(buf).cuda()[:, : rows * V].unflatten(1, (rows, V))


@pytest.mark.parametrize("logits", ["f32", "bf16"])
@pytest.mark.parametrize("V", VOCABS)
@pytest.mark.parametrize("top_k,top_p", [(1, 1.0), (40, 1.0), (1500, 1.0), (0, 0.9), (50, 0.9), (0, 0.3)])
def test_listed_rows_match_reference(logits, V, top_k, top_p):
    for B, gam in ((4, (3, 6)), (80, (3, 3))) if V == 4101 else ((4, (3, 6)),):
        inp, p, q, drafts = _inputs(V, logits, B, gam, 301 + V)
        say(f"listed rows {logits} V={V} B={B} top_k={top_k} top_p={top_p}")
        got = run_accept(None, None, drafts, inp.gamma, inp.u_acc, inp.u_res, p_dev=_padded(p), q_dev=_padded(q),
                         temperature=0.8, top_k=top_k, top_p=top_p)
        ref = oracle.accept_and_diverge(p, q, drafts, inp.gamma, inp.u_acc, inp.u_res, temperature=0.8, top_k=top_k,
                                        top_p=top_p)
        assert got["status"] == ref["status"] == 0
        nf, nb, nbm = _check_filtered(got, ref)
        say(f"  ok ({nf} filter-boundary skipped, {nb} boundary, {nbm} differ)")


@pytest.mark.parametrize("top_k,top_p", [(20, 1.0), (0, 0.9)])
def test_lists_over_several_launches(top_k, top_p):
    """More sequences than one launch takes: the lists' room is one launch's and
    is found cleared by the next, whose sequences are listed, swept or both."""
    V, B = 300, 4100
    inp, p, q, drafts = _inputs(V, "f32", B, (0, 2), 977)
    say(f"lists over two launches top_k={top_k} top_p={top_p}")
    bufs = sr.AcceptBuffers(B, p.shape[1] - 1, V, sr.SR_F32)
    args = (None, None, drafts, inp.gamma, inp.u_acc, inp.u_res)
    kw = dict(p_dev=_padded(p), q_dev=_padded(q), bufs=bufs, temperature=0.8, top_k=top_k, top_p=top_p)
    got = run_accept(*args, **kw)
    again = run_accept(*args, **kw)
    assert int((bufs.workspace != 0).sum()) == 0
    for k in ("accept_len", "out_tokens", "accept_prob", "kl", "tv"):
        np.testing.assert_array_equal(got[k], again[k], err_msg=k)
    seqs = list(range(0, 40)) + list(range(4080, 4100))
    sub = [np.asarray(x)[seqs] for x in (p, q, drafts, inp.gamma, inp.u_acc, inp.u_res)]
    ref = oracle.accept_and_diverge(*sub, temperature=0.8, top_k=top_k, top_p=top_p)
    assert got["status"] == ref["status"] == 0
    _check_filtered({k: v[seqs] if isinstance(v, np.ndarray) else v for k, v in got.items()}, ref)


LOWEST = {"f32": np.float32(-3.4028234663852886e38), "bf16": np.float32(-3.3895313892515355e38)}


@pytest.mark.parametrize("logits", ["f32", "bf16"])
@pytest.mark.parametrize("V", [60, 200, 4101])
@pytest.mark.parametrize("top_k,top_p", [(50, 1.0), (0, 0.9), (50, 0.9)])
def test_masks_of_the_lowest_value_match_reference(logits, V, top_k, top_p):
    """Most of the vocabulary masked with the type's lowest value rather than
    -inf (fewer entries left than top-k asks for, or just about as many):
    masked entries that the filter keeps have probability 0."""
    inp = level_inputs(small_shape(name=f"lowest-{logits}-{V}", B=4, V=V, gamma=(3, 5), seed=900 + V), kv=False)
    rng = np.random.default_rng(V)
    masked = rng.random(V) < (0.6 if V == 60 else 0.9)
    p, q = (np.where(masked, LOWEST[logits], x.astype(np.float32)) for x in (inp.p_logits, inp.q_logits))
    drafts = np.argmax(q + rng.gumbel(size=q.shape), axis=-1).astype(np.int32)
    if logits == "bf16":
        p, q = bf16_bits_from_f32(p), bf16_bits_from_f32(q)
    say(f"lowest {logits} V={V} top_k={top_k} top_p={top_p} ({int((~masked).sum())} entries not masked)")
    got = run_accept(None, None, drafts, inp.gamma, inp.u_acc, inp.u_res, p_dev=_padded(p), q_dev=_padded(q),
                     temperature=0.8, top_k=top_k, top_p=top_p)
    ref = oracle.accept_and_diverge(p, q, drafts, inp.gamma, inp.u_acc, inp.u_res, temperature=0.8, top_k=top_k,
                                    top_p=top_p)
    assert got["status"] == ref["status"] == 0
    _check_filtered(got, ref)


def _masked_rows(z, rng):
    """Reshape the rows by kind: what constrained decoding and flat models leave."""
    flat = z.reshape(-1, z.shape[-1])
    V = flat.shape[1]
    for i, row in enumerate(flat):
        kind = i % 7
        if kind == 1:  # the first half masked (a sample of the row's start sees nothing)
            row[: V // 2] = -np.inf
        elif kind == 2:  # three entries left
            row[rng.permutation(V)[3:]] = -np.inf
        elif kind == 3:  # 99% masked with a low but ordinary value
            row[rng.random(V) < 0.99] = -1.0e4
        elif kind == 4:  # two values
            row[:] = rng.integers(0, 2, V).astype(np.float32)
        elif kind == 5:  # one value
            row[:] = 3.0
        elif kind == 6:  # 97% masked, dealt in runs
            row[(np.arange(V) // 64) % 33 != 0] = -np.inf
    return z


@pytest.mark.parametrize("logits", ["f32", "bf16"])
@pytest.mark.parametrize("V,B", [(300, 6), (5003, 80), (50257, 6)])
@pytest.mark.parametrize("top_k,top_p", [(50, 1.0), (0, 0.9), (50, 0.9), (2000, 0.9), (4500, 1.0)])
def test_masked_and_tied_rows_match_reference(logits, V, B, top_k, top_p):
    """Rows with fewer entries than top-k asks for, and rows whose entries
    are mostly masks or equal, in both widths of the threshold kernel."""
    inp = level_inputs(small_shape(name=f"masked-{logits}-{V}", B=B, V=V, gamma=(3, 4), seed=700 + V), kv=False)
    rng = np.random.default_rng(V)
    p = _masked_rows(inp.p_logits.astype(np.float32).copy(), rng)
    q = _masked_rows(inp.q_logits.astype(np.float32).copy(), rng)
    drafts = np.argmax(q + rng.gumbel(size=q.shape), axis=-1).astype(np.int32)
    if logits == "bf16":
        p, q = bf16_bits_from_f32(p), bf16_bits_from_f32(q)
    say(f"masked rows {logits} V={V} B={B} top_k={top_k} top_p={top_p}")
    got = run_accept(None, None, drafts, inp.gamma, inp.u_acc, inp.u_res, p_dev=_padded(p), q_dev=_padded(q),
                     temperature=0.8, top_k=top_k, top_p=top_p)
    ref = oracle.accept_and_diverge(p, q, drafts, inp.gamma, inp.u_acc, inp.u_res, temperature=0.8, top_k=top_k,
                                    top_p=top_p)
    assert got["status"] == ref["status"] == 0
    _check_filtered(got, ref)


@pytest.mark.parametrize("logits", ["f32", "bf16"])
@pytest.mark.parametrize("top_k,top_p", [(50, 1.0), (0, 0.9), (50, 0.9)])
def test_lists_and_the_sweep_agree(logits, top_k, top_p):
    """A workspace of the bytes that a call needs at least, without room for
    lists, sends every row through the sweep, and one with room for short
    lists only those that keep more: the same decisions, and floats within the
    sweep's 32-bit sums of the lists' 64-bit ones (1e-6 of the value; 1e-7 near
    zero), but not the same bits: rows were listed. Each leaves the workspace
    all zero."""
    V, B = 33000, 12
    inp, p, q, drafts = _inputs(V, logits, B, (2, 5), 77)
    code = sr.SR_BF16 if logits == "bf16" else sr.SR_F32
    G = p.shape[1] - 1
    bufs = sr.AcceptBuffers(B, G, V, code)
    full = bufs.workspace
    nc = -(-V // 4096)  # records 32 B and four 8-byte sums per chunk; 24 bytes per row; aligned regions
    rows = B * (G + 1)
    up = lambda n: (n + 255) // 256 * 256  # noqa: E731
    least = up(rows * nc * 32) + up(rows * nc * 32) + up(rows * 16) + up(rows * 8) + 256
    lists = up((B + 1) * 4) + up(rows * 2 * 16)  # the swept positions and the rows' sums; then 2048 entries per row
    assert full.numel() == least + lists + rows * 2048 * 8
    args = (p, q, drafts, inp.gamma, inp.u_acc, inp.u_res)
    kw = dict(kv_len=inp.kv_len, temperature=0.8, top_k=top_k, top_p=top_p)
    a = run_accept(*args, bufs=bufs, **kw)
    assert int((full != 0).sum()) == 0
    for room in (0, lists + rows * 64 * 8):
        bufs.workspace = torch.zeros(least + room, dtype=torch.uint8, device="cuda")
        b = run_accept(*args, bufs=bufs, **kw)
        assert int((bufs.workspace != 0).sum()) == 0
        for k in ("accept_len", "out_tokens", "new_len", "status"):
            np.testing.assert_array_equal(a[k], b[k], err_msg=k)
        for k in ("accept_prob", "p_tok", "q_tok", "kl", "tv"):
            np.testing.assert_allclose(a[k], b[k], rtol=1e-6, atol=1e-7, err_msg=k)
        if room == 0:
            assert any((a[k] != b[k])[~np.isnan(a[k])].any() for k in ("kl", "tv"))
    bufs.workspace = torch.zeros(least - 256, dtype=torch.uint8, device="cuda")
    with pytest.raises(RuntimeError):
        run_accept(*args, bufs=bufs, **kw)
