"""The C-ABI boundary on the host (CPU only): the library loads, exports every
declared entry point, sizes workspaces, and rejects bad arguments with the
documented codes before anything reaches the GPU."""
import ctypes
import os
import re

import pytest

import paper_2607_05439_amd as dcp

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
FAKE = 0x10000  # a 256-byte aligned non-null address; never dereferenced on these paths


def declared_functions():
    src = open(os.path.join(ROOT, "include", "dcp.h")).read()
    src = re.sub(r"/\*.*?\*/", "", src, flags=re.S)
    return sorted(set(re.findall(r"\b(dcp_[a-z_]+)\s*\(", src)))


def test_exports_every_declared_symbol():
    names = declared_functions()
    assert set(names) == set(dcp.EXPORTS)
    lib = dcp.lib()
    for n in names:
        assert hasattr(lib, n), n
    assert "gfx950" in dcp.dcp_version()


def shape(**kw):
    base = dict(n_tokens=24000, c_s=384, c_z=128, n_heads=16, head_dim=24, act_dtype=dcp.DCP_BF16,
                out_dtype=dcp.DCP_F32, ln_eps=1e-5)
    base.update(kw)
    return dcp.make_shape(**base)


def weights():
    return dcp.make_weights(FAKE, FAKE, FAKE, FAKE, FAKE)


def attention(sh, w=None, s=FAKE, z=FAKE, q_row0=0, n_q=24000, n_kb=6, out=FAKE, ws=FAKE, ws_bytes=1 << 40):
    return dcp.lib().dcp_pair_bias_attention(ctypes.byref(sh), ctypes.byref(w or weights()), s, z, None, q_row0, n_q,
                                             n_kb, out, ws, ws_bytes, None)


def test_workspace_sizes():
    big = dcp.dcp_workspace_size(shape(), 24000, 6)
    # q, k, v tiles (3 x 16 x 24000 x 32 x 2 B) + gate + 6 partials: a few hundred MB
    assert 200e6 < big < 400e6
    assert dcp.dcp_workspace_size(shape(), 0, 6) == 0
    small = dcp.dcp_workspace_size(shape(n_tokens=128, c_s=128, c_z=32, n_heads=4, head_dim=32,
                                         act_dtype=dcp.DCP_F32), 128, 4)
    assert 0 < small < 2e6
    # more key blocks need more partial storage
    assert dcp.dcp_workspace_size(shape(), 24000, 12) > big


def test_workspace_bytes_matches_status_form():
    """dcp_workspace_bytes (the size-returning query) agrees with
    dcp_workspace_size on valid shapes and is 0, with a message, on bad ones."""
    cases = [(shape(), 24000, 6), (shape(), 24000, 1), (shape(), 3000, 4), (shape(n_tokens=12000), 3000, 4),
             (shape(n_tokens=1024), 1024, 4), (shape(n_tokens=4800), 4800, 10), (shape(n_tokens=1), 1, 1),
             (shape(n_tokens=128, c_s=128, c_z=32, n_heads=4, head_dim=32, act_dtype=dcp.DCP_F32), 128, 4),
             (shape(n_tokens=50, c_s=40, c_z=64, n_heads=4, head_dim=16), 40, 3)]
    for sh, n_q, n_kb in cases:
        got = dcp.dcp_workspace_bytes(sh, n_q, n_kb)
        assert got == dcp.dcp_workspace_size(sh, n_q, n_kb) > 0
        assert dcp.dcp_last_error() == ""
    assert dcp.dcp_workspace_bytes(shape(), 0, 6) == 0
    assert dcp.dcp_last_error() == ""
    bad = [(None, 10, 1), (shape(n_tokens=0), 10, 1), (shape(c_z=512), 10, 1), (shape(n_heads=32), 10, 1),
           (shape(ln_eps=float("nan")), 10, 1), (shape(), -1, 1), (shape(), 24001, 1), (shape(), 100, 0),
           (shape(), 100, 24001), (shape(n_tokens=0), 0, 1)]
    for sh, n_q, n_kb in bad:
        assert dcp.dcp_workspace_bytes(sh, n_q, n_kb) == 0
        assert len(dcp.dcp_last_error()) > 0


@pytest.mark.parametrize("kw,code", [
    (dict(n_tokens=0), dcp.DCP_ERR_INVALID_ARGUMENT),
    (dict(c_z=0), dcp.DCP_ERR_INVALID_ARGUMENT),
    (dict(act_dtype=7), dcp.DCP_ERR_INVALID_ARGUMENT),
    (dict(ln_eps=-1.0), dcp.DCP_ERR_INVALID_ARGUMENT),
    (dict(ln_eps=float("nan")), dcp.DCP_ERR_INVALID_ARGUMENT),
    (dict(c_z=512), dcp.DCP_ERR_UNSUPPORTED),
    (dict(n_heads=32), dcp.DCP_ERR_UNSUPPORTED),
    (dict(head_dim=100, n_heads=1), dcp.DCP_ERR_UNSUPPORTED),
    (dict(c_s=5000), dcp.DCP_ERR_UNSUPPORTED),
])
def test_bad_shapes(kw, code):
    sh = shape(**kw)
    assert attention(sh) == code
    assert len(dcp.dcp_last_error()) > 0
    out = ctypes.c_size_t()
    assert dcp.lib().dcp_workspace_size(ctypes.byref(sh), 100, 1, ctypes.byref(out)) == code


def test_bad_ranges():
    E = dcp.DCP_ERR_INVALID_ARGUMENT
    sh = shape()
    assert attention(sh, n_q=-1) == E
    assert attention(sh, q_row0=-1, n_q=10) == E
    assert attention(sh, q_row0=23990, n_q=11) == E
    assert attention(sh, n_kb=0) == E
    assert attention(sh, n_kb=24001) == E
    assert attention(sh, s=0) == E
    assert attention(sh, z=0) == E
    assert attention(sh, out=0) == E
    assert attention(sh, z=FAKE + 2) == E  # misaligned
    w = dcp.make_weights(FAKE, FAKE, 0, FAKE, FAKE)
    assert attention(sh, w=w) == E
    # the fused path reads w_b and ln_gamma with 16-byte loads
    assert attention(sh, w=dcp.make_weights(FAKE, FAKE, FAKE, FAKE, FAKE + 4)) == E
    assert "w_b" in dcp.dcp_last_error()
    assert attention(sh, w=dcp.make_weights(FAKE, FAKE, FAKE, FAKE, FAKE, ln_gamma=FAKE + 8)) == E
    assert dcp.lib().dcp_pair_bias_attention(None, ctypes.byref(weights()), FAKE, FAKE, None, 0, 1, 1, FAKE, FAKE,
                                             1 << 40, None) == E


def partial(sh, k0=0, k1=4000, m=FAKE, l=FAKE, acc=FAKE, gate=0, ws=FAKE, ws_bytes=1 << 40, n_q=24000):
    return dcp.lib().dcp_pair_bias_attention_partial(ctypes.byref(sh), ctypes.byref(weights()), FAKE, FAKE, None, 0,
                                                     n_q, k0, k1, m, l, acc, gate, ws, ws_bytes, None)


def test_partial_rejections():
    E = dcp.DCP_ERR_INVALID_ARGUMENT
    sh = shape()
    assert partial(sh, k0=-1) == E
    assert partial(sh, k0=10, k1=9) == E
    assert partial(sh, k1=24001) == E
    assert partial(sh, m=0) == E and "m_out" in dcp.dcp_last_error()
    assert partial(sh, acc=0) == E
    assert partial(sh, m=FAKE + 2) == E  # misaligned
    need = dcp.dcp_workspace_size(sh, 24000, 1)
    assert partial(sh, ws_bytes=need - 1) == dcp.DCP_ERR_WORKSPACE
    assert partial(sh, n_q=0, ws=0, ws_bytes=0) == dcp.DCP_OK
    assert dcp.lib().dcp_pair_bias_attention_partial(None, ctypes.byref(weights()), FAKE, FAKE, None, 0, 1, 0, 1, FAKE,
                                                     FAKE, FAKE, 0, FAKE, 1 << 40, None) == E
    assert partial(shape(c_z=100), ws_bytes=1 << 40) == dcp.DCP_ERR_UNSUPPORTED


def test_bad_workspace():
    sh = shape()
    need = dcp.dcp_workspace_size(sh, 24000, 6)
    assert attention(sh, ws_bytes=need - 1) == dcp.DCP_ERR_WORKSPACE
    assert attention(sh, ws=0) == dcp.DCP_ERR_WORKSPACE
    assert attention(sh, ws=FAKE + 128) == dcp.DCP_ERR_WORKSPACE
    assert "workspace" in dcp.dcp_last_error()


def test_empty_stripe_is_ok_without_touching_the_gpu():
    assert attention(shape(), q_row0=24000, n_q=0, ws=0, ws_bytes=0) == dcp.DCP_OK


def test_bias_project_rejections():
    L = dcp.lib()
    sh, w = shape(), weights()
    E = dcp.DCP_ERR_INVALID_ARGUMENT
    assert L.dcp_bias_project(ctypes.byref(sh), ctypes.byref(w), FAKE, 4, 8, 8 * 128 - 1, FAKE, None) == E
    assert L.dcp_bias_project(ctypes.byref(sh), ctypes.byref(w), 0, 4, 8, 1024, FAKE, None) == E
    assert L.dcp_bias_project(ctypes.byref(sh), ctypes.byref(w), FAKE, -1, 8, 1024, FAKE, None) == E
    assert L.dcp_bias_project(ctypes.byref(sh), ctypes.byref(w), FAKE, 0, 8, 1024, FAKE, None) == dcp.DCP_OK
    for wb in (dcp.make_weights(FAKE, FAKE, FAKE, FAKE, FAKE + 4), dcp.make_weights(0, 0, 0, 0, FAKE, ln_gamma=FAKE + 4),
               dcp.make_weights(0, 0, 0, 0, FAKE, ln_beta=FAKE + 8)):
        assert L.dcp_bias_project(ctypes.byref(sh), ctypes.byref(wb), FAKE, 4, 8, 1024, FAKE, None) == E
    bad = shape(c_z=1000)
    assert L.dcp_bias_project(ctypes.byref(bad), ctypes.byref(w), FAKE, 4, 8, 8000, FAKE, None) == \
        dcp.DCP_ERR_UNSUPPORTED


def test_block_merge_rejections():
    L = dcp.lib()
    E = dcp.DCP_ERR_INVALID_ARGUMENT
    assert L.dcp_block_merge(0, 4, 2, 3, FAKE, FAKE, FAKE, None, None, None, None, FAKE, 0, None) == E
    assert L.dcp_block_merge(2, 4, 2, 3, 0, FAKE, FAKE, None, None, None, None, FAKE, 0, None) == E
    assert L.dcp_block_merge(2, 4, 2, 3, FAKE, FAKE, FAKE, None, None, None, None, FAKE, 9, None) == E
    assert L.dcp_block_merge(2, 4, 64, 128, FAKE, FAKE, FAKE, None, None, None, None, FAKE, 0, None) == \
        dcp.DCP_ERR_UNSUPPORTED
    assert L.dcp_block_merge(2, 0, 2, 3, FAKE, FAKE, FAKE, None, None, None, None, FAKE, 0, None) == dcp.DCP_OK


def test_timing_events_pairing():
    assert dcp.lib().dcp_set_timing_events(FAKE, None) == dcp.DCP_ERR_INVALID_ARGUMENT
    assert dcp.lib().dcp_set_timing_events(None, None) == dcp.DCP_OK


def test_binding_raises():
    with pytest.raises(dcp.DcpError) as e:
        dcp.dcp_workspace_size(shape(n_heads=0), 10, 1)
    assert e.value.code == dcp.DCP_ERR_INVALID_ARGUMENT


# ----------------------------------------------------------------------------- sparse atom attention
def sparse_shape(**kw):
    base = dict(n_atoms=96000, c_atom=128, c_ap=16, n_heads=4, head_dim=32, k=128, act_dtype=dcp.DCP_BF16,
                out_dtype=dcp.DCP_F32, p_gathered=0, ln_eps=1e-5)
    base.update(kw)
    return dcp.make_sparse_shape(**base)


def sparse(sh, w=None, a=FAKE, p=FAKE, nbr=FAKE, q_row0=0, n_q=24000, n_kb=4, out=FAKE, ws=FAKE, ws_bytes=1 << 40):
    return dcp.lib().dcp_sparse_pair_bias_attention(ctypes.byref(sh), ctypes.byref(w or weights()), a, p, nbr, q_row0,
                                                    n_q, n_kb, out, ws, ws_bytes, None)


def test_sparse_workspace_sizes():
    # q, g fp32 for 24000 queries + K, V bf16 for 96000 atoms
    got = dcp.dcp_sparse_workspace_size(sparse_shape(), 24000)
    assert got >= 2 * 24000 * 128 * 4 + 2 * 96000 * 128 * 2
    assert got < 1.01 * (2 * 24000 * 128 * 4 + 2 * 96000 * 128 * 2) + 4096
    f32 = dcp.dcp_sparse_workspace_size(sparse_shape(act_dtype=dcp.DCP_F32), 24000)
    assert f32 > got
    assert dcp.dcp_sparse_workspace_size(sparse_shape(), 0) == 0


@pytest.mark.parametrize("kw,code", [
    (dict(n_atoms=0), dcp.DCP_ERR_INVALID_ARGUMENT),
    (dict(k=0), dcp.DCP_ERR_INVALID_ARGUMENT),
    (dict(act_dtype=3), dcp.DCP_ERR_INVALID_ARGUMENT),
    (dict(p_gathered=2), dcp.DCP_ERR_INVALID_ARGUMENT),
    (dict(ln_eps=float("inf")), dcp.DCP_ERR_INVALID_ARGUMENT),
    (dict(n_heads=8), dcp.DCP_ERR_UNSUPPORTED),
    (dict(head_dim=16), dcp.DCP_ERR_UNSUPPORTED),
    (dict(c_ap=32), dcp.DCP_ERR_UNSUPPORTED),
    (dict(k=257), dcp.DCP_ERR_UNSUPPORTED),
    (dict(n_atoms=5_000_000), dcp.DCP_ERR_UNSUPPORTED),
    (dict(c_atom=100), dcp.DCP_ERR_UNSUPPORTED),  # bf16 needs a multiple of 32
])
def test_sparse_bad_shapes(kw, code):
    sh = sparse_shape(**kw)
    assert sparse(sh) == code
    assert len(dcp.dcp_last_error()) > 0
    out = ctypes.c_size_t()
    assert dcp.lib().dcp_sparse_workspace_size(ctypes.byref(sh), 100, ctypes.byref(out)) == code


def test_sparse_bad_arguments():
    E, W = dcp.DCP_ERR_INVALID_ARGUMENT, dcp.DCP_ERR_WORKSPACE
    sh = sparse_shape()
    assert sparse(sh, q_row0=-1) == E
    assert sparse(sh, q_row0=80000) == E      # 80000 + 24000 > 96000
    assert sparse(sh, n_q=-1) == E
    assert sparse(sh, n_kb=0) == E
    assert sparse(sh, n_kb=96001) == E
    assert sparse(sh, a=None) == E
    assert sparse(sh, p=None) == E
    assert sparse(sh, nbr=None) == E
    assert sparse(sh, out=None) == E
    assert sparse(sh, a=FAKE + 8) == E        # misaligned
    assert sparse(sh, nbr=FAKE + 2) == E
    assert sparse(sh, w=dcp.make_weights(FAKE, FAKE, FAKE, FAKE, None)) == E
    assert sparse(sh, ws=None) == W
    assert sparse(sh, ws=FAKE + 16) == W
    assert sparse(sh, ws_bytes=1000) == W
    # an f32 call accepts any c_atom and unaligned weights
    assert sparse(sparse_shape(act_dtype=dcp.DCP_F32, c_atom=100), ws_bytes=1000) == W
    assert sparse(sh, n_q=0, ws=None) == dcp.DCP_OK  # no-op


# ----------------------------------------------------------------------------- k nearest neighbours
def knn(x_q=FAKE, n_q=100, x_c=FAKE, n_c=1000, c0=0, self0=-1, gq=None, gc=None, mode=0, k=128, idx=FAKE, d2=FAKE,
        ws=FAKE, ws_bytes=1 << 20):
    return dcp.lib().dcp_knn_topk(x_q, n_q, x_c, n_c, c0, self0, gq, gc, mode, k, idx, d2, ws, ws_bytes, None)


def test_knn_bad_arguments():
    E, U = dcp.DCP_ERR_INVALID_ARGUMENT, dcp.DCP_ERR_UNSUPPORTED
    assert knn(k=0) == E
    assert knn(k=257) == U
    assert knn(n_q=-1) == E
    assert knn(n_c=-1) == E
    assert knn(c0=-1) == E
    assert knn(c0=2**31 - 100, n_c=1000) == E     # indices past int32
    assert knn(mode=3) == E
    assert knn(mode=1) == E                        # groups required
    assert knn(x_q=None) == E
    assert knn(x_c=None) == E
    assert knn(idx=None) == E
    assert knn(x_q=FAKE + 2) == E                  # misaligned
    W = dcp.DCP_ERR_WORKSPACE
    assert knn(ws=None) == W
    assert knn(ws=FAKE + 16) == W                  # not 256-byte aligned
    assert knn(ws_bytes=dcp.dcp_knn_workspace_size(1000) - 1) == W
    assert knn(n_q=0) == dcp.DCP_OK                # no-op
    assert len(dcp.dcp_last_error()) == 0


def test_knn_workspace_size():
    # 16 bytes per candidate (rounded to 256) plus 32 per started 128
    assert dcp.dcp_knn_workspace_size(0) == 0
    assert dcp.dcp_knn_workspace_size(1) == 256 + 32
    assert dcp.dcp_knn_workspace_size(128) == 2048 + 32
    assert dcp.dcp_knn_workspace_size(129) == 2304 + 64
    assert dcp.dcp_knn_workspace_size(96000) == 96000 * 16 + 750 * 32
    rc = dcp.lib().dcp_knn_workspace_size(-1, ctypes.byref(ctypes.c_size_t()))
    assert rc == dcp.DCP_ERR_INVALID_ARGUMENT


def test_topk_merge_bad_arguments():
    E = dcp.DCP_ERR_INVALID_ARGUMENT
    L = dcp.lib()
    assert L.dcp_topk_merge(10, 0, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, None) == E
    assert L.dcp_topk_merge(10, 300, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, None) == dcp.DCP_ERR_UNSUPPORTED
    assert L.dcp_topk_merge(-1, 8, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, None) == E
    assert L.dcp_topk_merge(10, 8, FAKE, None, FAKE, FAKE, FAKE, FAKE, None) == E
    assert L.dcp_topk_merge(0, 8, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, None) == dcp.DCP_OK


# ----------------------------------------------------------------------------- pair transition
def trans(n=1000, c_z=128, hidden=512, dt=dcp.DCP_BF16, eps=1e-5, w=FAKE, zi=FAKE, zo=FAKE * 64, ws=FAKE * 4,
          ws_bytes=1 << 30):
    return dcp.lib().dcp_pair_transition(n, c_z, hidden, dt, ctypes.c_float(eps), w, w, w, None, None, zi, zo, ws,
                                         ws_bytes, None)


def test_transition_arguments():
    E, U, W = dcp.DCP_ERR_INVALID_ARGUMENT, dcp.DCP_ERR_UNSUPPORTED, dcp.DCP_ERR_WORKSPACE
    assert 390_000 < dcp.dcp_transition_workspace_size(128, 512, dcp.DCP_BF16) < 400_000
    assert dcp.dcp_transition_workspace_size(64, 100, dcp.DCP_F32) == 0
    assert trans(c_z=64) == U                    # bf16 needs 128 / 512
    assert trans(hidden=256) == U
    assert trans(dt=dcp.DCP_F32, c_z=300) == U
    assert trans(dt=dcp.DCP_F32, hidden=2048) == U
    assert trans(dt=5) == E
    assert trans(c_z=0) == E
    assert trans(n=-1) == E
    assert trans(eps=-1.0) == E
    assert trans(w=None) == E
    assert trans(zi=None) == E
    assert trans(zi=FAKE + 8) == E               # misaligned
    assert trans(zi=FAKE, zo=FAKE + 256) == E    # overlapping, not equal
    assert trans(ws=None) == W
    assert trans(ws_bytes=1000) == W
    assert trans(n=0, ws=None) == dcp.DCP_OK


# ----------------------------------------------------------------------------- atom -> token mean
def test_scatter_mean_arguments():
    E, U, W = dcp.DCP_ERR_INVALID_ARGUMENT, dcp.DCP_ERR_UNSUPPORTED, dcp.DCP_ERR_WORKSPACE
    assert dcp.dcp_scatter_mean_workspace_size(24000, 128) >= 24000 * 128 * 8 + 24000 * 4
    L = dcp.lib()
    ok = lambda **kw: L.dcp_scatter_mean(kw.get("na", 100), kw.get("nt", 10), kw.get("c", 128), kw.get("di", 1),
                                         kw.get("do", 0), kw.get("a", FAKE), kw.get("idx", FAKE), kw.get("out", FAKE),
                                         kw.get("ws", FAKE), kw.get("wsb", 1 << 30), None)
    assert ok(c=0) == E
    assert ok(c=513) == U
    assert ok(na=-1) == E
    assert ok(di=4) == E
    assert ok(a=None) == E
    assert ok(idx=None) == E
    assert ok(out=None) == E
    assert ok(idx=FAKE + 2) == E
    assert ok(ws=None) == W
    assert ok(wsb=100) == W
    assert ok(nt=0, out=None, ws=None) == dcp.DCP_OK


def test_noalloc_rejects_beyond_its_scratch():
    """dcp_pair_bias_attention_noalloc checks sizes before anything else: a
    call needing more than DCP_NOALLOC_SCRATCH_BYTES is refused on the host
    (here without a GPU), bad arguments get their usual codes."""
    assert dcp.NOALLOC_SCRATCH_BYTES == 128 << 20
    lib = dcp.lib()

    def call(sh, n_q, n_kb, q_row0=0):
        return lib.dcp_pair_bias_attention_noalloc(ctypes.byref(sh), ctypes.byref(weights()), FAKE, FAKE, None,
                                                   q_row0, n_q, n_kb, FAKE, None)

    need = dcp.dcp_workspace_size(shape(), 24000, 6)
    assert need > dcp.NOALLOC_SCRATCH_BYTES
    assert call(shape(), 24000, 6) == dcp.DCP_ERR_WORKSPACE
    msg = dcp.dcp_last_error()
    assert "maximum" in msg and str(need) in msg
    assert call(shape(n_tokens=0), 10, 1) == dcp.DCP_ERR_INVALID_ARGUMENT
    assert call(shape(), 100, 0) == dcp.DCP_ERR_INVALID_ARGUMENT
    assert call(shape(c_z=512), 10, 1) == dcp.DCP_ERR_UNSUPPORTED
    # the workloads it is meant for fit: a 1024-token layer, a 3000-row stripe of 12000 tokens
    assert dcp.dcp_workspace_size(shape(n_tokens=1024), 1024, 4) <= dcp.NOALLOC_SCRATCH_BYTES
    assert dcp.dcp_workspace_size(shape(n_tokens=12000), 3000, 4) <= dcp.NOALLOC_SCRATCH_BYTES


def test_layout_probes_check_the_librarys_own_helpers():
    """The lane-layout probes compile against the library's device header: every helper they check
    is defined there, none in the probes themselves, where it would be code that only a test runs."""
    probe = open(os.path.join(ROOT, "tests", "probes", "probe.hip")).read()
    header = open(os.path.join(ROOT, "paper_2607_05439_amd", "csrc", "cdna4.h")).read()
    define = r"__device__\s+__forceinline__\s+[\w ]+?\b(\w+)\("
    assert re.findall(define, probe) == []
    used = [n for n in re.findall(define, header) if re.search(rf"\b{n}(<\d+>)?\(", probe)]
    assert set(used) >= {"mfma32", "mfma16", "swap32", "swap16", "sum4", "max4", "transpose_bias", "dma_b128"}
