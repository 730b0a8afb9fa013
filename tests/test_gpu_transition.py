"""Pair transition (LayerNorm + SwiGLU + residual) on the GPU against the fp64
oracle, through the C-ABI (GPU)."""
import numpy as np
import pytest

import oracle
import synth
from gpu_helpers import DCP_BF16, DCP_F32, log, rel_err

pytestmark = pytest.mark.gpu


def dev(a):
    import torch
    a = np.ascontiguousarray(a)
    if a.dtype == np.uint16:
        return torch.from_numpy(a.view(np.int16)).view(torch.bfloat16).to("cuda:0")
    return torch.from_numpy(a).to("cuda:0")


def run(z, w, dtype, n_pairs=None, in_place=False, eps=1e-5):
    """dcp_pair_transition on device tensor z (flattened pairs); returns the output tensor."""
    import torch
    import paper_2607_05439_amd as dcp
    c_z = z.shape[-1]
    hidden = w["w1"].shape[0]
    n = z.numel() // c_z if n_pairs is None else n_pairs
    ws_bytes = dcp.dcp_transition_workspace_size(c_z, hidden, dtype)
    ws = torch.empty(max(ws_bytes, 256), dtype=torch.uint8, device="cuda:0")
    out = z if in_place else torch.empty_like(z)
    W = {k: (None if v is None else dev(v)) for k, v in w.items()}
    dcp.dcp_pair_transition(n, c_z, hidden, dtype, eps, W["w1"], W["w2"], W["w3"], W["gamma"], W["beta"], z, out,
                            ws, ws.numel())
    return out


def host_f64(t):
    import torch
    return t.float().cpu().numpy().astype(np.float64)


def test_f32_whole_output():
    wl, hidden = synth.transition_workload("trans40_f32")
    z = synth.z_host(wl, range(wl.n_tok))  # [40, 40, 32] fp32
    for affine in (False, True):
        w = synth.transition_weights(wl, hidden, affine=affine)
        ref = oracle.transition(z, w["w1"], w["w2"], w["w3"], w["gamma"], w["beta"])
        zt = dev(z)
        got = host_f64(run(zt, w, DCP_F32))
        err = rel_err(got, ref)
        log(f"case trans40_f32 affine={affine}: rel err {err:.3e}")
        assert err <= 1e-5
        inplace = run(zt, w, DCP_F32, in_place=True)
        assert np.array_equal(host_f64(inplace), got)


def test_bf16_whole_output():
    wl, hidden = synth.transition_workload("trans192_bf16")
    z = synth.z_host(wl, range(wl.n_tok))  # [192, 192, 128] bf16 bits
    for affine in (False, True):
        w = synth.transition_weights(wl, hidden, affine=affine)
        ref = oracle.transition(z, w["w1"], w["w2"], w["w3"], w["gamma"], w["beta"])
        got = host_f64(run(dev(z), w, DCP_BF16))
        err = rel_err(got, ref)
        log(f"case trans192_bf16 affine={affine}: rel err {err:.3e}")
        assert err <= 1e-2


def test_bf16_ragged_inplace_deterministic():
    """Pair counts that are not a multiple of the 256-pair group, in place
    against out of place, repeated calls, and pairs past n_pairs untouched."""
    import torch
    wl, hidden = synth.transition_workload("trans192_bf16")
    z = synth.z_host(wl, range(8))  # 8 rows x 192 pairs
    w = synth.transition_weights(wl, hidden, affine=True)
    flat = z.reshape(-1, 128)
    for n in (1, 255, 257, 1000, len(flat)):
        ref = oracle.transition(flat[:n], w["w1"], w["w2"], w["w3"], w["gamma"], w["beta"])
        zt = dev(flat)
        a = run(zt, w, DCP_BF16, n_pairs=n)
        b = run(zt, w, DCP_BF16, n_pairs=n)
        assert torch.equal(a[:n], b[:n])
        err = rel_err(host_f64(a[:n]), ref)
        assert err <= 1e-2, (n, err)
        zc = zt.clone()
        run(zc, w, DCP_BF16, n_pairs=n, in_place=True)
        assert torch.equal(zc[:n], a[:n])
        assert torch.equal(zc[n:], zt[n:])
    run(dev(flat), w, DCP_BF16, n_pairs=0)


@pytest.mark.parametrize("n", [1, 16, 17, 31, 33, 16383, 16384, 16385])
def test_bf16_split_kernel_edges(n):
    """Pair counts around the 16-pair tiles and 32-pair workgroups of the kernel
    for few pairs, and on both sides of the rule that chooses it: against the
    oracle (bf16 operands and output: the 1e-2 bound), in place, the pairs past
    n untouched."""
    import torch
    wl, hidden = synth.transition_workload("trans192_bf16")
    w = synth.transition_weights(wl, hidden, affine=True)
    flat = synth.z_host(wl, range(n // 192 + 1)).reshape(-1, 128)
    zt = dev(flat)
    got = run(zt, w, DCP_BF16, n_pairs=n)
    some = np.unique(np.r_[np.arange(min(n, 64)), np.arange(max(0, n - 300), n)])
    ref = oracle.transition(flat[some], w["w1"], w["w2"], w["w3"], w["gamma"], w["beta"])
    assert rel_err(host_f64(got[torch.from_numpy(some).to("cuda:0")]), ref) <= 1e-2
    zc = zt.clone()
    run(zc, w, DCP_BF16, n_pairs=n, in_place=True)
    assert torch.equal(zc[:n], got[:n])
    assert torch.equal(zc[n:], zt[n:])


@pytest.mark.parametrize("n", [1, 31, 1000, 8192, 16384])
def test_bf16_chunks_match_the_whole_call(n):
    """Pairs have the same bits whichever kernel the size of the call chooses: a tensor processed in
    chunks is the tensor processed at once, in place or not."""
    import torch
    wl, hidden = synth.transition_workload("trans192_bf16")
    w = synth.transition_weights(wl, hidden, affine=True)
    zt = dev(synth.z_host(wl, range(192)).reshape(-1, 128))
    whole = run(zt, w, DCP_BF16)
    for r in sorted({0, 7 * n, len(zt) - n} & set(range(len(zt) - n + 1))):
        part = zt[r:r + n].clone()
        assert torch.equal(run(part, w, DCP_BF16, n_pairs=n), whole[r:r + n])
        run(part, w, DCP_BF16, n_pairs=n, in_place=True)
        assert torch.equal(part, whole[r:r + n])


def test_bf16_full_size_in_place_sampled():
    """The 24000-token pair tensor (147 GB, bf16) updated in place in one call,
    as the benchmark does; sampled pairs against the oracle on the generator's
    host copy of the same values."""
    import torch
    wl, hidden = synth.transition_workload("trans24000_bf16")
    n = wl.n_tok
    log("allocating and generating z for asm24000_bf16 (147 GB)")
    z = torch.empty((n, n, 128), dtype=torch.bfloat16, device="cuda:0")
    synth.z_fill_device(wl, z.data_ptr(), 0, n, torch.cuda.current_stream().cuda_stream)
    w = synth.transition_weights(wl, hidden)
    log("case trans24000_bf16 in place")
    run(z, w, DCP_BF16, in_place=True)
    rng = np.random.default_rng(0)
    rows = [0, 1, 12345, n - 1]
    cols = np.concatenate([[0, 1, 255, 256, n - 1], rng.choice(n, 300, replace=False)])
    zh = synth.z_host(wl, rows)[:, cols]  # [4, len(cols), 128]
    ref = oracle.transition(zh, w["w1"], w["w2"], w["w3"])
    got = host_f64(z[rows][:, torch.from_numpy(cols).to("cuda:0")])
    err = rel_err(got, ref)
    log(f"  {zh.shape[0] * zh.shape[1]} pairs rel err {err:.3e}")
    assert err <= 1e-2
    del z
    torch.cuda.empty_cache()


@pytest.mark.parametrize("c_z,hidden", [(4, 16), (20, 48), (32, 128), (64, 80), (100, 400), (128, 512), (132, 16),
                                        (256, 1024), (30, 64), (32, 72)])
def test_f32_widths_and_tile_edges(c_z, hidden):
    """fp32 widths on both kernels (c_z a multiple of 4 and hidden of 16, or
    not) and every template width, pair counts around the 16- and 32-pair tiles
    and the rule between them; a weight off 16-byte alignment gives the vector
    kernel's result. Tolerance: the fp32 acceptance bound (1e-5 of the largest
    value), far above sqrt(hidden) * 2^-24."""
    import torch
    rng = np.random.default_rng(c_z * 1000 + hidden)
    w = {"w1": rng.standard_normal((hidden, c_z)) / np.sqrt(c_z), "w2": rng.standard_normal((hidden, c_z)) / np.sqrt(c_z),
         "w3": rng.standard_normal((c_z, hidden)) / np.sqrt(hidden), "gamma": 1 + 0.25 * rng.standard_normal(c_z),
         "beta": 0.25 * rng.standard_normal(c_z)}
    w = {k: v.astype(np.float32) for k, v in w.items()}
    for n in (1, 15, 17, 33) + ((4096, 4097, 12288, 12289) if c_z == 32 else ()):
        z = rng.standard_normal((n, c_z)).astype(np.float32)
        ref = oracle.transition(z, w["w1"], w["w2"], w["w3"], w["gamma"], w["beta"])
        zt = dev(z)
        got = run(zt, w, DCP_F32)
        assert rel_err(host_f64(got), ref) <= 1e-5
        assert torch.equal(run(zt.clone(), w, DCP_F32, in_place=True), got)
    import paper_2607_05439_amd as dcp
    off = torch.empty(hidden * c_z + 1, device="cuda:0")
    off[1:] = dev(w["w1"]).reshape(-1)
    out = torch.empty_like(zt)
    W = {k: dev(v) for k, v in w.items()}
    dcp.dcp_pair_transition(n, c_z, hidden, DCP_F32, 1e-5, off[1:], W["w2"], W["w3"], W["gamma"], W["beta"], zt, out,
                            None, 0)
    assert rel_err(host_f64(out), ref) <= 1e-5


@pytest.mark.parametrize("c_z,hidden", [(32, 128), (100, 400), (128, 512), (256, 64)])
def test_f32_chunks_match_the_whole_call(c_z, hidden):
    """One tile of 16 pairs per workgroup or two, by the size of the call: the same bits."""
    import torch
    rng = np.random.default_rng(c_z)
    w = {"w1": rng.standard_normal((hidden, c_z)), "w2": rng.standard_normal((hidden, c_z)),
         "w3": rng.standard_normal((c_z, hidden)), "gamma": rng.standard_normal(c_z), "beta": rng.standard_normal(c_z)}
    w = {k: v.astype(np.float32) for k, v in w.items()}
    z = dev(rng.standard_normal((4200, c_z)).astype(np.float32))
    whole = run(z, w, DCP_F32)
    for r, n in ((0, 4096), (100, 4097), (4199, 1), (7, 1000)):
        assert torch.equal(run(z[r:r + n].clone(), w, DCP_F32), whole[r:r + n])


@pytest.mark.parametrize("c_z,hidden", [(20, 48), (32, 128), (100, 400), (132, 16)])
@pytest.mark.parametrize("name", ["w1", "w2"])
def test_f32_infinite_weight(c_z, hidden, name):
    """An infinite weight of W1 or W2 in the last channel: the outputs it reaches are infinite (the
    products with the finite others are not 0), none is NaN."""
    rng = np.random.default_rng(c_z)
    w = {"w1": 0.1 + 0.2 * rng.random((hidden, c_z)), "w2": 0.1 + 0.2 * rng.random((hidden, c_z)),
         "w3": 0.1 + 0.2 * rng.random((c_z, hidden)), "gamma": np.full(c_z, 0.1), "beta": np.ones(c_z)}
    w = {k: v.astype(np.float32) for k, v in w.items()}  # LN z = 1 + 0.1 (..) > 0: every product is positive
    w[name][hidden - 1, c_z - 1] = np.inf
    z = rng.uniform(-1, 1, (40, c_z)).astype(np.float32)
    got = host_f64(run(dev(z), w, DCP_F32))
    assert np.all(got == np.inf)
