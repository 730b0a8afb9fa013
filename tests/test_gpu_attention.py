"""dcp_pair_bias_attention through the C-ABI against the fp64 oracle (GPU).

Tolerances (max|err| / max|ref|): 1e-5 for fp32 inputs, 1e-2 for bf16 inputs,
1e-6 between blocked and unblocked GPU results with fp32 output.
"""
import numpy as np
import pytest

import synth
from gpu_helpers import DCP_BF16, DCP_F32, Device, check_partitions, log, rel_err, sample_rows, workload

pytestmark = pytest.mark.gpu

TOL_F32, TOL_BF16, TOL_BLOCKED = 1e-5, 1e-2, 1e-6


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return torch


def _np(t):
    return t.float().cpu().numpy().astype(np.float64)


# ----------------------------------------------------------------------------- tiny fp32 (general path)
def test_tiny128_f32_parity(torch_cuda):
    log("case tiny128_f32 n_kb=1")
    d = Device(workload("tiny128_f32"))
    rows = np.arange(128)
    ref = d.oracle_rows(rows)
    got = _np(d.attention(0, 128, 1))
    err = rel_err(got, ref)
    log(f"  rel err {err:.3e}")
    assert err <= TOL_F32


def test_tiny128_f32_blocked(torch_cuda):
    log("case tiny128_f32 n_kb=4 vs 1")
    d = Device(workload("tiny128_f32"))
    a = _np(d.attention(0, 128, 1))
    b = _np(d.attention(0, 128, 4))
    assert rel_err(b, a) <= TOL_BLOCKED
    assert rel_err(b, d.oracle_rows(np.arange(128), n_blocks=4)) <= TOL_F32


def test_general_path_bf16_inputs(torch_cuda):
    log("case general path, bf16 inputs, c_z=64 H=4 d=16, masked, stripe")
    wl = workload(n_tok=50, c_s=40, c_z=64, n_heads=4, head_dim=16, dtype="bf16", mask="random:7")
    d = Device(wl)
    got = _np(d.attention(3, 40, 3))
    ref = d.oracle_rows(np.arange(3, 43))
    assert rel_err(got, ref) <= TOL_F32


@pytest.mark.parametrize("n_tok,c_s,c_z,h,d,dtype,n_kb", [
    # the tiled kernel: every head layout, pair widths at and between its templates, key tiles
    # of 16 over 4 waves (1, 15, 17, 64, 65 keys), rows on both sides of the one-pass rule (256)
    (1, 16, 16, 1, 4, "f32", 1), (15, 33, 32, 3, 12, "f32", 2), (17, 128, 48, 4, 32, "f32", 3),
    (64, 64, 64, 5, 16, "f32", 1), (65, 70, 96, 8, 16, "bf16", 5), (100, 128, 112, 16, 8, "f32", 4),
    (90, 36, 128, 9, 8, "bf16", 1), (255, 128, 128, 4, 32, "f32", 3), (257, 96, 32, 4, 16, "f32", 3),
    # two rows per workgroup (at most 32 channels, 512 rows and parts), an odd row count
    (515, 32, 32, 4, 32, "f32", 1), (131, 32, 16, 6, 12, "bf16", 4),
    # shapes it does not take: the general kernel
    (40, 20, 24, 2, 6, "f32", 3), (33, 128, 144, 2, 64, "f32", 2), (260, 48, 40, 10, 12, "bf16", 2)])
def test_general_path_shapes(torch_cuda, n_tok, c_s, c_z, h, d, dtype, n_kb):
    """Whole layers of the general path with an affine LayerNorm, masked keys whose s and z hold
    NaN, and the ranges of a ring; the fp32 acceptance bound."""
    log(f"case general path N={n_tok} c_s={c_s} c_z={c_z} H={h} d={d} {dtype} n_kb={n_kb}")
    n_mask = n_tok // 7
    wl = workload(n_tok=n_tok, c_s=c_s, c_z=c_z, n_heads=h, head_dim=d, dtype=dtype,
                  mask=f"random:{n_mask}" if n_mask else "none")
    dv = Device(wl, affine=True)
    rows = np.arange(n_tok) if dv.mask_host is None else np.flatnonzero(dv.mask_host)
    ref = dv.oracle_rows(rows)
    if n_mask:
        masked = torch_cuda.from_numpy(dv.mask_host == 0).cuda()
        dv.z[:, masked] = float("nan")
        dv.s[masked] = float("nan")
    got = _np(dv.attention(0, n_tok, n_kb))[rows]
    assert rel_err(got, ref) <= TOL_F32
    assert rel_err(_np(dv.attention(0, n_tok, 1))[rows], got) <= TOL_BLOCKED
    assert np.array_equal(_np(dv.attention(0, n_tok, n_kb))[rows], got)
    if n_tok >= 256 and c_z % 16 == 0:  # the tiled kernel: one part here, three in stripes of few rows
        clean = Device(wl, affine=True)  # no NaN in the masked tokens' own rows
        check_partitions(clean, 0, n_tok, clean.attention(0, n_tok, n_kb), n_kb=3)
    if n_tok > 20:  # a stripe, bf16 output
        sub = rows[(rows >= 3) & (rows < n_tok - 2)]
        out = _np(dv.attention(3, n_tok - 5, n_kb, out_dtype=DCP_BF16))[sub - 3]
        assert rel_err(out, ref[np.isin(rows, sub)]) <= TOL_BF16


@pytest.mark.parametrize("n_tok,n_kb,c_z,h,d", [(40, 1, 32, 4, 32), (131, 3, 128, 8, 16), (300, 1, 64, 16, 8),
                                                (601, 1, 32, 4, 16), (33, 2, 24, 2, 6)])
def test_general_path_infinite_value(torch_cuda, n_tok, n_kb, c_z, h, d):
    """v of one output overflows to +inf at the last key (a part's last, off the 16-key tiles): that
    output is +inf in every row, none is NaN, and the others are what they are without it."""
    log(f"case general path, infinite v at key {n_tok - 1} of {n_tok}, n_kb={n_kb} c_z={c_z} H={h} d={d}")
    wl = workload(n_tok=n_tok, c_s=64, c_z=c_z, n_heads=h, head_dim=d, dtype="f32")
    s = synth.s_host(wl).copy()
    s[:, 0] = 0.0
    s[-1, 0] = 1e30
    dv = Device(wl, affine=True, s_override=s)
    for name in ("w_q", "w_k", "w_v", "w_g"):
        dv.w_host[name] = dv.w_host[name].copy()
        dv.w_host[name][:, 0] = 0.0
    ref = dv.oracle_rows(np.arange(n_tok))
    dv.w_host["w_v"][5, 0] = 1e30
    for name in ("w_q", "w_k", "w_v", "w_g"):
        dv.w[name] = torch_cuda.from_numpy(np.ascontiguousarray(dv.w_host[name])).to(dv.dev)
    got = _np(dv.attention(0, n_tok, n_kb))
    assert np.all(got[:, 5] == np.inf)
    rest = np.arange(h * d) != 5
    assert rel_err(got[:, rest], ref[:, rest]) <= TOL_F32


# ----------------------------------------------------------------------------- fused bf16 path
def test_pad1024_parity(torch_cuda):
    log("case pad1024_bf16 n_kb=4 f32 out")
    d = Device(workload("pad1024_bf16"))
    ref = d.oracle_rows(np.arange(1024))
    got = _np(d.attention(0, 1024, 4))
    err = rel_err(got, ref)
    log(f"  rel err {err:.3e}")
    assert err <= TOL_BF16
    got_bf = _np(d.attention(0, 1024, 4, out_dtype=DCP_BF16))
    assert rel_err(got_bf, ref) <= TOL_BF16


def test_pad1024_blocked_vs_unblocked(torch_cuda):
    log("case pad1024_bf16 blocked vs unblocked")
    d = Device(workload("pad1024_bf16"))
    a = _np(d.attention(0, 1024, 1))
    for nb in (4, 7, 64):
        b = _np(d.attention(0, 1024, nb))
        err = rel_err(b, a)
        log(f"  n_kb={nb} rel diff {err:.3e}")
        assert err <= TOL_BLOCKED
    check_partitions(d, 0, 1024, d.attention(0, 1024, 4))


def test_deterministic(torch_cuda):
    log("case pad1024_bf16 repeat")
    d = Device(workload("pad1024_bf16"))
    a = d.attention(0, 1024, 4)
    b = d.attention(0, 1024, 4)
    assert torch_cuda.equal(a, b)


def test_masked_keys_never_read(torch_cuda):
    log("case pad1024_bf16 masked z perturbed")
    d = Device(workload("pad1024_bf16"))
    a = d.attention(0, 1024, 4)
    masked = np.flatnonzero(d.mask_host == 0)
    z2 = d.z.clone()
    z2[:, masked, :] = 1000.0
    b = d.attention(0, 1024, 4, z=z2)
    assert torch_cuda.equal(a, b)


def test_affine_constants_irrelevant(torch_cuda):
    log("case beta and b_b change nothing")
    wl = workload(n_tok=96, mask="tail:5")
    d = Device(wl, affine=True)
    a = _np(d.attention(0, 96, 2))
    b = _np(d.attention(0, 96, 2, drop_affine=True))
    assert rel_err(a, b) <= TOL_BLOCKED
    assert rel_err(a, d.oracle_rows(np.arange(96))) <= TOL_BF16


@pytest.mark.parametrize("n_tok,q_row0,n_q,n_kb,mask", [
    (1, 0, 1, 1, "none"),
    (5, 1, 3, 2, "none"),
    (16, 0, 16, 1, "none"),
    (17, 0, 17, 17, "tail:1"),
    (37, 5, 19, 3, "random:6"),
    (100, 60, 40, 5, "random:30"),
    (333, 0, 333, 2, "tail:13"),
    # few query rows over many keys: the launch splits the keys into many short
    # parts of whole 16-key tiles, whatever the key blocks
    (2048, 100, 50, 1, "random:200"),
    (1500, 0, 64, 3, "tail:7"),
])
def test_ragged_and_small(torch_cuda, n_tok, q_row0, n_q, n_kb, mask):
    log(f"case ragged N={n_tok} q_row0={q_row0} n_q={n_q} n_kb={n_kb} mask={mask}")
    d = Device(workload(n_tok=n_tok, mask=mask))
    got = _np(d.attention(q_row0, n_q, n_kb))[:n_q]
    ref = d.oracle_rows(np.arange(q_row0, q_row0 + n_q))
    err = rel_err(got, ref)
    log(f"  rel err {err:.3e}")
    assert err <= TOL_BF16


def test_all_keys_masked_gives_zero(torch_cuda):
    log("case all keys masked")
    wl = workload(n_tok=40)
    d = Device(wl, mask=np.zeros(40, np.uint8))
    out = d.attention(0, 40, 3)
    assert torch_cuda.count_nonzero(out).item() == 0
    wl32 = workload(n_tok=20, c_s=16, c_z=8, n_heads=2, head_dim=4, dtype="f32")
    d32 = Device(wl32, mask=np.zeros(20, np.uint8))
    assert torch_cuda.count_nonzero(d32.attention(0, 20, 2)).item() == 0


def test_one_block_entirely_masked(torch_cuda):
    log("case a whole key block masked")
    m = np.ones(200, np.uint8)
    m[50:100] = 0  # block 1 of 4
    d = Device(workload(n_tok=200), mask=m)
    got = _np(d.attention(0, 200, 4))
    assert rel_err(got, d.oracle_rows(np.arange(200))) <= TOL_BF16
    assert rel_err(got, _np(d.attention(0, 200, 1))) <= TOL_BLOCKED
    check_partitions(d, 0, 200, d.attention(0, 200, 4))


def test_n_q_zero_is_noop(torch_cuda):
    import paper_2607_05439_amd as dcp
    d = Device(workload(n_tok=32))
    shape = d.shape()
    assert dcp.dcp_workspace_size(shape, 0, 1) == 0
    out = torch_cuda.full((1, 384), 7.0, device="cuda")
    dcp.dcp_pair_bias_attention(shape, d.weights(), d.s, d.z, None, 32, 0, 1, out, None, 0, None)
    torch_cuda.cuda.synchronize()
    assert torch_cuda.all(out == 7.0)


# ----------------------------------------------------------------------------- larger workloads, sampled rows
def test_ico4800_sampled(torch_cuda):
    wl = workload("ico4800_bf16")
    log("case ico4800_bf16 n_kb=10 sampled rows")
    d = Device(wl)
    got = _np(d.attention(0, wl.n_tok, wl.n_key_blocks))
    rows = sample_rows(wl.n_tok, wl.stripes, wl.n_key_blocks, 96, d.mask_host)
    err = rel_err(got[rows], d.oracle_rows(rows))
    log(f"  {len(rows)} rows rel err {err:.3e}")
    assert err <= TOL_BF16


def test_grid12000_stripes_sampled(torch_cuda):
    wl = workload("grid12000_bf16")
    log("case grid12000_bf16 4 stripes x 4 key blocks, sampled rows")
    d = Device(wl)
    for q0, nq in wl.stripes:
        got = _np(d.attention(q0, nq, wl.n_key_blocks))
        rows = sample_rows(wl.n_tok, [(q0, nq)], 1, 24, None, seed=q0)
        rows = [r for r in rows if q0 <= r < q0 + nq]
        err = rel_err(got[np.array(rows) - q0], d.oracle_rows(rows))
        log(f"  stripe {q0}: {len(rows)} rows rel err {err:.3e}")
        assert err <= TOL_BF16


@pytest.mark.parametrize("n_tok,q_row0,n_q,n_kb", [(1, 0, 1, 1), (16, 0, 16, 16), (47, 30, 17, 2), (130, 1, 1, 130),
                                                   (1100, 1083, 17, 9), (1100, 500, 33, 1000), (2050, 7, 40, 64)])
def test_part_partition_edges(torch_cuda, n_tok, q_row0, n_q, n_kb):
    """Row tiles and key parts at their edges: one row, one key, parts of one 16-key tile, more key
    blocks than tiles, a last tile of a few keys; against the oracle, and one block against many."""
    log(f"case N={n_tok} rows {q_row0}+{n_q} n_kb={n_kb}")
    m = np.ones(n_tok, np.uint8)
    m[5:n_tok - 1:11] = 0
    d = Device(workload(n_tok=n_tok), mask=m)
    got = _np(d.attention(q_row0, n_q, n_kb))
    assert rel_err(got, d.oracle_rows(np.arange(q_row0, q_row0 + n_q))) <= TOL_BF16
    assert rel_err(_np(d.attention(q_row0, n_q, 1)), got) <= TOL_BLOCKED
    assert np.array_equal(_np(d.attention(q_row0, n_q, n_kb)), got)
    if n_tok > 1000:
        whole = d.attention(0, n_tok, 1)  # its rows are split into fewer parts
        assert not torch_cuda.equal(whole[q_row0:q_row0 + n_q], d.attention(q_row0, n_q, n_kb))
        assert rel_err(_np(whole[q_row0:q_row0 + n_q]), got) <= TOL_BLOCKED


@pytest.mark.parametrize("n_tok,c_z,h,d,dtype,q_row0,n_q,n_kb", [
    (100, 128, 16, 24, "bf16", 0, 100, 1), (100, 128, 16, 24, "bf16", 40, 20, 3), (1400, 128, 16, 24, "bf16", 500, 200, 1),
    (40, 32, 4, 32, "f32", 0, 40, 1), (70, 128, 8, 16, "f32", 0, 70, 3), (300, 32, 4, 16, "f32", 0, 300, 2),
    (70, 24, 2, 6, "f32", 0, 70, 1), (70, 24, 2, 6, "f32", 0, 70, 4)])
def test_nan_of_an_unmasked_pair_or_token_propagates(torch_cuda, n_tok, c_z, h, d, dtype, q_row0, n_q, n_kb):
    """A NaN in one pair vector makes its row NaN and no other; one in the s of a key makes every row
    that attends to it NaN; in a call and in partial states merged, whichever part the key lies in."""
    import paper_2607_05439_amd as dcp
    log(f"case NaN: N={n_tok} c_z={c_z} H={h} d={d} {dtype} rows {q_row0}+{n_q} n_kb={n_kb}")
    wl = workload(n_tok=n_tok, c_s=64, c_z=c_z, n_heads=h, head_dim=d, dtype=dtype)
    m = np.ones(n_tok, np.uint8)
    m[2::5] = 0
    dv = Device(wl, mask=m)
    key, row = n_tok - 1 - (m[-1] == 0), n_q // 2
    clean = dv.attention(q_row0, n_q, n_kb)

    def states_merged():
        shape, f32 = dv.shape(), dict(dtype=torch_cuda.float32, device="cuda:0")
        ms, ls = (torch_cuda.empty((2, h, n_q), **f32) for _ in range(2))
        acc, gate = torch_cuda.empty((2, n_q, h * d), **f32), torch_cuda.empty((n_q, h * d), **f32)
        ws = torch_cuda.empty(dcp.dcp_workspace_size(shape, n_q, 1), dtype=torch_cuda.uint8, device="cuda:0")
        cut, z_ptr = n_tok - 4, dv.z.data_ptr() + q_row0 * n_tok * c_z * dv.z.element_size()
        for i, (k0, k1) in enumerate(((0, cut), (cut, n_tok))):
            dcp.dcp_pair_bias_attention_partial(shape, dv.weights(), dv.s, z_ptr, dv.mask, q_row0, n_q, k0, k1, ms[i],
                                                ls[i], acc[i], gate, ws, ws.numel())
        out = torch_cuda.empty((n_q, h * d), **f32)
        dcp.dcp_block_merge(2, n_q, h, d, ms, ls, acc, None, None, None, gate, out, DCP_F32)
        return out

    merged = states_merged()
    dv.z[q_row0 + row, key, 3] = float("nan")
    for got, ref in ((dv.attention(q_row0, n_q, n_kb), clean), (states_merged(), merged)):
        assert got[row].isnan().all()
        others = np.arange(n_q) != row
        assert torch_cuda.equal(got[others], ref[others])
    dv.s[key, 1] = float("nan")
    assert dv.attention(q_row0, n_q, n_kb).isnan().all()
    assert states_merged().isnan().all()
