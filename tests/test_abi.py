"""The C ABI without a GPU: the library loads, exports every symbol the
headers declare, and rejects malformed descriptors with the documented
error codes before any device work (validation is host-only)."""

import ctypes
import math
import os
import random
import re

import pytest

from paper_2406_14898_amd import flglm as F

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _lib():
    if not os.path.exists(F.LIB_PATH):
        from paper_2406_14898_amd import build
        build.build()
    return F.load()


def _declared():
    names = set()
    for h in ("flglm.h", "flglm_testing.h"):
        src = open(os.path.join(ROOT, "include", h)).read()
        names |= set(re.findall(r"^\s*(?:const\s+char\s*\*|int)\s+(fl_\w+)\s*\(", src, re.M))
    return names


def test_exports_every_declared_symbol():
    lib = _lib()
    decl = _declared()
    assert len(decl) >= 17
    assert decl == set(F.EXPORTS)
    for n in decl:
        assert hasattr(lib, n), n


def test_stack_desc_accepts_the_glm_block():
    _lib()
    h = F.fl_stack_create(F.stack_desc(2, 256, 4, 1024, 32, F.FL_BF16, residual_alpha=7.48, rotary_2d=True,
                                       num_prefix=16))
    F.fl_stack_destroy(h)


def _tiny_handle(dtype=F.FL_BF16):
    _lib()
    return F.fl_stack_create(F.stack_desc(2, 256, 4, 1024, 32, dtype))


@pytest.mark.parametrize("desc,code", [
    (dict(hidden=250), F.FL_ERR_SHAPE), (dict(num_heads=3), F.FL_ERR_SHAPE),
    (dict(num_heads=8), F.FL_ERR_SHAPE),  # head dim 32
    (dict(ffn_hidden=1000), F.FL_ERR_SHAPE), (dict(rotary_dim=48), F.FL_ERR_SHAPE),
    (dict(rotary_dim=96), F.FL_ERR_SHAPE), (dict(num_layers=0), F.FL_ERR_SHAPE),
    (dict(dtype=7), F.FL_ERR_SHAPE), (dict(ln_eps=0.0), F.FL_ERR_SHAPE),
    (dict(rope_base=0.0), F.FL_ERR_SHAPE), (dict(hidden=4352, num_heads=34), F.FL_ERR_SHAPE),
    (dict(num_prefix=-1), F.FL_ERR_SHAPE), (dict(num_prefix=4097), F.FL_ERR_SHAPE),
    (dict(num_prefix=16, dtype=F.FL_F32), F.FL_ERR_SHAPE),       # the prefix path is bf16 only
    (dict(residual_alpha=-1.0), F.FL_ERR_SHAPE), (dict(residual_alpha=float("inf")), F.FL_ERR_SHAPE),
    (dict(rotary_2d=True, rotary_dim=64), F.FL_ERR_SHAPE),       # 2-D positions need rotary = head dim / 2
])
def test_stack_desc_validation(desc, code):
    _lib()
    base = dict(num_layers=2, hidden=256, num_heads=4, ffn_hidden=1024, rotary_dim=32, dtype=F.FL_BF16)
    base.update(desc)
    with pytest.raises(F.FlglmError) as e:
        F.fl_stack_create(F.stack_desc(**base))
    assert e.value.code == code


@pytest.mark.parametrize("cu,csp,pre,code", [
    ([0], [0], None, F.FL_ERR_SEQLENS),                      # empty batch: no sequences, no tokens
    ([0, 3], [0], None, F.FL_ERR_CLIENTS),                   # no clients
    ([0, 3, 3, 7], [0, 1, 3], None, F.FL_ERR_SEQLENS),      # empty sequence
    ([1, 3, 7], [0, 1, 2], None, F.FL_ERR_SEQLENS),         # cu[0] != 0
    ([0, 3, 7], [0, 2, 2], None, F.FL_ERR_CLIENTS),         # client without sequences
    ([0, 3, 7], [0, 1, 3], None, F.FL_ERR_CLIENTS),         # csp[C] != S
    ([0, 3, 7], [1, 2], None, F.FL_ERR_CLIENTS),            # csp[0] != 0
    ([0, 3, 7], [0, 1, 2], [0, 5], F.FL_ERR_PREFIX),        # prefix longer than its sequence
    ([0, 3, 7], [0, 1, 2], [-1, 2], F.FL_ERR_PREFIX),
])
def test_batch_validation(cu, csp, pre, code):
    h = _tiny_handle()
    b = F.BatchDesc(cu, csp, pre)
    with pytest.raises(F.FlglmError) as e:
        F.fl_stack_workspace_bytes(h, b, False)
    assert e.value.code == code
    F.fl_stack_destroy(h)


def test_batch_validation_totals():
    h = _tiny_handle()
    b = F.BatchDesc([0, 3, 7], [0, 1, 2])
    b.desc.total_tokens = 8
    with pytest.raises(F.FlglmError) as e:
        F.fl_stack_saved_bytes(h, b, False)
    assert e.value.code == F.FL_ERR_SEQLENS
    b = F.BatchDesc([0, 3, 7], [0, 1, 2], max_seqlen=5)
    with pytest.raises(F.FlglmError) as e:
        F.fl_stack_saved_bytes(h, b, False)
    assert e.value.code == F.FL_ERR_SEQLENS
    F.fl_stack_destroy(h)


def test_client_token_range_host_only():
    _lib()
    b = F.BatchDesc([0, 3, 8, 12, 20], [0, 2, 3, 4])
    assert F.fl_client_token_range(b, 0) == (0, 8)
    assert F.fl_client_token_range(b, 1) == (8, 12)
    assert F.fl_client_token_range(b, 2) == (12, 20)
    with pytest.raises(F.FlglmError) as e:
        F.fl_client_token_range(b, 3)
    assert e.value.code == F.FL_ERR_ARG


def test_sizes_scale_with_tokens_and_recompute():
    h = _tiny_handle()
    b1 = F.BatchDesc([0, 64, 128], [0, 1, 2])
    b2 = F.BatchDesc([0, 128, 256], [0, 1, 2])
    s1 = F.fl_stack_saved_bytes(h, b1, False)
    s2 = F.fl_stack_saved_bytes(h, b2, False)
    r1 = F.fl_stack_saved_bytes(h, b1, True)
    assert s2 > s1 > r1 > 0
    # recompute keeps only the inputs of blocks 2..N: (N-1) * T * H * 2 bytes
    assert r1 == 1 * 128 * 256 * 2
    assert F.fl_stack_workspace_bytes(h, b2, False) > F.fl_stack_workspace_bytes(h, b1, False)
    F.fl_stack_destroy(h)


def test_forward_rejects_before_any_device_work():
    """Bad arguments are caught on the host: no stream, no device memory
    needed to get the error codes."""
    h = _tiny_handle()
    b = F.BatchDesc([0, 64, 128], [0, 1, 2])
    ws_n = F.fl_stack_workspace_bytes(h, b, False)
    L = F.fl_layer_params(*([16] * 12))
    lib = F.load()
    arr = (F.fl_layer_params * 2)(L, L)
    # NULL x
    rc = lib.fl_server_stack_forward(h, ctypes.byref(b.desc), arr, None, 4096, None, 0, 1 << 20, ws_n, None)
    assert rc == F.FL_ERR_NULL
    # misaligned y
    rc = lib.fl_server_stack_forward(h, ctypes.byref(b.desc), arr, 1 << 30, (1 << 31) + 4, None, 0, 1 << 34, ws_n,
                                     None)
    assert rc == F.FL_ERR_ALIGN
    # overlapping x / y
    rc = lib.fl_server_stack_forward(h, ctypes.byref(b.desc), arr, 1 << 30, (1 << 30) + 4096, None, 0, 1 << 34,
                                     ws_n, None)
    assert rc == F.FL_ERR_ALIAS
    # workspace too small
    rc = lib.fl_server_stack_forward(h, ctypes.byref(b.desc), arr, 1 << 30, 1 << 31, None, 0, 1 << 34, ws_n - 1,
                                     None)
    assert rc == F.FL_ERR_WORKSPACE
    # NULL parameter pointer
    bad = (F.fl_layer_params * 2)(L, F.fl_layer_params(*([16] * 11 + [0])))
    rc = lib.fl_server_stack_forward(h, ctypes.byref(b.desc), bad, 1 << 30, 1 << 31, None, 0, 1 << 34, ws_n, None)
    assert rc == F.FL_ERR_NULL
    assert "NULL" in F.fl_last_error()
    # backward: dx overlapping dy
    G = F.fl_layer_grads(*([16] * 12))
    garr = (F.fl_layer_grads * 2)(G, G)
    rc = lib.fl_server_stack_backward(h, ctypes.byref(b.desc), arr, garr, 1 << 30, 1 << 35, 1 << 31, 1 << 31, 0,
                                      1 << 34, ws_n, None)
    assert rc == F.FL_ERR_ALIAS
    F.fl_stack_destroy(h)


def test_adam_and_average_reject_before_any_device_work():
    """The server-update entry points validate on the host (fake device
    addresses are never dereferenced when validation fails)."""
    lib = _lib()
    A, B, C, D, E = 1 << 30, 1 << 31, 3 << 30, 1 << 32, 5 << 30
    n = 1 << 20
    adam = lambda p=A, g=B, m=C, v=D, p16=None, n=n, step=1, lr=2e-2, b1=0.9, b2=0.999, eps=1e-8, zg=0: \
        lib.fl_adam_step(p, g, m, v, p16, n, step, lr, b1, b2, eps, zg, None)
    assert adam(p=None) == F.FL_ERR_NULL
    assert adam(v=None) == F.FL_ERR_NULL
    assert adam(g=B + 4) == F.FL_ERR_ALIGN
    assert adam(p16=E + 8) == F.FL_ERR_ALIGN
    assert adam(m=A + 16) == F.FL_ERR_ALIAS
    assert adam(p16=D + 4 * n - 16) == F.FL_ERR_ALIAS
    assert adam(step=0) == F.FL_ERR_ARG
    assert adam(n=-1) == F.FL_ERR_ARG
    assert adam(lr=-1.0) == F.FL_ERR_ARG
    assert adam(lr=float("nan")) == F.FL_ERR_ARG
    assert adam(b1=1.0) == F.FL_ERR_ARG
    assert adam(b2=-0.1) == F.FL_ERR_ARG
    assert adam(eps=-1e-8) == F.FL_ERR_ARG
    assert adam(zg=2) == F.FL_ERR_ARG
    assert adam(n=0) == F.FL_OK  # no-op, nothing launched

    def avg(ptrs, ptrs16=None, n=n):
        arr = (ctypes.c_void_p * len(ptrs))(*ptrs)
        arr16 = None if ptrs16 is None else (ctypes.c_void_p * len(ptrs16))(*ptrs16)
        return lib.fl_average_replicas(len(ptrs), arr, arr16, n, None)

    assert lib.fl_average_replicas(0, None, None, n, None) == F.FL_ERR_ARG
    assert lib.fl_average_replicas(1, None, None, n, None) == F.FL_ERR_NULL
    assert avg([A + (i << 28) for i in range(33)]) == F.FL_ERR_ARG
    assert avg([A, None]) == F.FL_ERR_NULL
    assert avg([A, B], [C, None]) == F.FL_ERR_NULL
    assert avg([A, B + 4]) == F.FL_ERR_ALIGN
    assert avg([A, A + 16]) == F.FL_ERR_ALIAS
    assert avg([A, B], [C, A + 4 * n - 16]) == F.FL_ERR_ALIAS
    assert avg([A, B], n=-5) == F.FL_ERR_ARG
    assert avg([A, B], n=0) == F.FL_OK


def test_client_handle_validation_host_only():
    """Client-side entry points: descriptor checks at create, id and label
    checks on the host before anything is enqueued."""
    lib = _lib()
    for vocab, hidden, dt in ((100, 256, F.FL_BF16), (1000, 200, F.FL_BF16), (1000, 256, 9), (0, 256, F.FL_F32)):
        with pytest.raises(F.FlglmError) as e:
            F.fl_client_create(vocab, hidden, dt)
        assert e.value.code == F.FL_ERR_SHAPE
    h = F.fl_client_create(1000, 256, F.FL_BF16)
    ws_n = F.fl_client_workspace_bytes(h, 10)
    assert ws_n >= 10 * 1024 * 2  # padded logits
    assert F.fl_client_workspace_bytes(h, 20) > ws_n
    ids = (ctypes.c_int32 * 10)(*([5] * 9 + [1000]))
    WS, OUT, TAB = 1 << 34, 1 << 30, 1 << 32
    rc = lib.fl_embedding_forward(h, TAB, ids, 10, OUT, WS, ws_n, None)
    assert rc == F.FL_ERR_ARG and "token id" in F.fl_last_error()
    rc = lib.fl_embedding_backward(h, ids, 10, OUT, TAB, WS, ws_n, None)
    assert rc == F.FL_ERR_ARG
    rc = lib.fl_embedding_forward(h, TAB, ids, 10, OUT, WS, ws_n - 1, None)
    assert rc == F.FL_ERR_WORKSPACE
    rc = lib.fl_embedding_forward(h, TAB + 8, ids, 10, OUT, WS, ws_n, None)
    assert rc == F.FL_ERR_ALIGN
    labels = (ctypes.c_int32 * 10)(*([-100] * 9 + [1000]))
    lt, ls = 1 << 31, (1 << 31) + 4096
    rc = lib.fl_lm_head_forward(h, OUT, None, None, TAB, labels, 10, lt, ls, WS, ws_n, None)
    assert rc == F.FL_ERR_ARG and "label" in F.fl_last_error()
    rc = lib.fl_lm_head_forward(h, OUT, None, None, TAB, labels, 10, WS + 256, ls, WS, ws_n, None)
    assert rc == F.FL_ERR_ALIAS
    ok_labels = (ctypes.c_int32 * 10)(*([-100] * 10))
    rc = lib.fl_lm_head_forward(h, OUT, TAB + (1 << 20), None, TAB, ok_labels, 10, lt, ls, WS, ws_n, None)
    assert rc == F.FL_ERR_NULL and "both or neither" in F.fl_last_error()
    rc = lib.fl_lm_head_backward(h, OUT, None, TAB, 10, ctypes.c_float(float("inf")), lt, None, None, None, WS,
                                 ws_n, None)
    assert rc == F.FL_ERR_ARG
    rc = lib.fl_lm_head_backward(h, OUT, None, TAB, 0, ctypes.c_float(1.0), lt, None, None, None, WS, ws_n, None)
    assert rc == F.FL_ERR_ARG
    rc = lib.fl_lm_head_backward(h, OUT, None, TAB, 10, ctypes.c_float(1.0), lt, lt + (1 << 20), lt + (1 << 21),
                                 None, WS, ws_n, None)
    assert rc == F.FL_ERR_ARG and "without a final LayerNorm" in F.fl_last_error()
    F.fl_client_destroy(h)


def test_missing_library_raises_instead_of_falling_back():
    """Without the built HIP library every entry point raises: there is no
    CPU path to fall back on (fresh interpreter, library path pointed at a
    file that does not exist)."""
    import subprocess
    import sys
    import textwrap
    code = textwrap.dedent('''
        import sys
        from paper_2406_14898_amd import flglm as F, ServerStack
        F.load.__defaults__ = ("/nonexistent/libflglm.so",)
        try:
            ServerStack(2, 256, 4, 1024, 32, dtype="f32")
        except F.FlglmError as e:
            print("RAISED", e)
            sys.exit(0)
        sys.exit(3)
    ''')
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", code], cwd=root, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "HIP library not built" in r.stdout


def test_noalloc_forward_rejects_what_does_not_fit():
    """The allocation-free forward's limits are checked on the host before
    anything else: a batch larger than the static scratch array, or with more
    sequences than its kernel-argument plan holds."""
    _lib()
    h = F.fl_stack_create(F.stack_desc(1, 4096, 32, 16384, 64, F.FL_BF16))
    L = F.fl_layer_params(*([256] * 12))
    with pytest.raises(F.FlglmError) as e:
        F.fl_server_stack_forward_noalloc(h, F.BatchDesc([0, 4000], [0, 1]), [L], 1 << 40, 1 << 41, 0)
    assert e.value.code == F.FL_ERR_WORKSPACE and "scratch" in str(e.value)
    many = list(range(F.FL_NOALLOC_MAX_SEQS + 2))
    with pytest.raises(F.FlglmError) as e:
        F.fl_server_stack_forward_noalloc(h, F.BatchDesc(many, [0, F.FL_NOALLOC_MAX_SEQS + 1]), [L], 1 << 40,
                                          1 << 41, 0)
    assert e.value.code == F.FL_ERR_ARG
    # a batch that fits: rejected only for the NULL output (still no device work)
    with pytest.raises(F.FlglmError) as e:
        F.fl_server_stack_forward_noalloc(h, F.BatchDesc([0, 1000], [0, 1]), [L], 1 << 40, None, 0)
    assert e.value.code == F.FL_ERR_NULL
    F.fl_stack_destroy(h)


@pytest.mark.parametrize("seed", range(6))
def test_attention_ds_tiles_count_visible_tile_pairs(seed):
    """The stored softmax gradient holds one 64 x 64 tile per (query tile, key
    tile) pair with at least one visible pair (the oracle's mask), plus the
    prefix key tiles every query tile meets, per head: the size the library
    asks for equals that brute-force count (host-only)."""
    import numpy as np
    import oracle
    _lib()
    rng = np.random.default_rng(seed)
    S = int(rng.integers(1, 6))
    lens = rng.integers(1, 300, S)
    if seed == 0:
        lens[:] = [64, 128, 1, 65, 192][:S] if S <= 5 else lens
    prefix = None if seed % 2 else rng.integers(0, lens + 1).astype(np.int32)
    nh, num_prefix = int(rng.integers(1, 4)), int(rng.choice([0, 1, 64, 70]))
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    ntp = (num_prefix + 63) // 64
    tiles = 0
    for s in range(S):
        L = int(lens[s])
        m = oracle.allowed_mask(L, None if prefix is None else int(prefix[s]))
        nt = (L + 63) // 64
        for qt in range(nt):
            tiles += ntp
            for kt in range(nt):
                tiles += bool(m[64 * qt:64 * qt + 64, 64 * kt:64 * kt + 64].any())
    off_bytes = ((S + 1) * 8 + 255) // 256 * 256
    assert F.fl_test_attention_ds_bytes(cu, prefix, nh, num_prefix) == off_bytes + nh * tiles * 64 * 64 * 2


def test_host_tensors_are_refused_before_the_library():
    """Every tensor argument is device memory: a host tensor raises FL_ERR_ARG
    in the binding, so no host address ever reaches a kernel."""
    import torch
    with pytest.raises(F.FlglmError) as e:
        F._ptr(torch.zeros(4))
    assert e.value.code == F.FL_ERR_ARG
    assert F._ptr(None) is None and F._ptr(4096) == 4096


@pytest.mark.parametrize("layout", [F.FL_GEMM_NT, F.FL_GEMM_NN, F.FL_GEMM_TN])
def test_gemm_plans_cover_the_product(layout):
    """The launches that the bf16 GEMM's planner chooses (host code): over any
    shape, scratch and column sums asked for or not, they cover every row once,
    a first launch ends at a whole tile (at a whole 256-row block where column
    sums are formed), slices have at least two stages (weight gradients:
    of the tiles past whole rounds only) and their fp32 sums fit the scratch."""
    rng = random.Random(layout)
    two = sliced = 0
    for _ in range(3000):
        M = int(math.exp(rng.uniform(0, math.log(60000))))
        N, K = 256 * rng.randint(1, 64), 64 * int(math.exp(rng.uniform(0, math.log(256))))
        if layout == F.FL_GEMM_TN:
            M, K = 256 * rng.randint(1, 64), int(math.exp(rng.uniform(0, math.log(60000))))
        part = rng.choice((0, 1 << 20, 64 << 20))
        sums = layout == F.FL_GEMM_NN and rng.random() < 0.5
        plan = F.fl_test_gemm_plan(layout, M, N, K, part, sums)
        what = (layout, M, N, K, part, sums, plan)
        assert 1 <= len(plan) <= 2 and sum(p[0] for p in plan) == M and all(p[0] > 0 for p in plan), what
        stages = (K + 63) // 64
        for rows, tile, slices in plan:
            assert tile in ((64, 128, 256) if layout == F.FL_GEMM_TN else (64, 128, 192, 256)), what
            assert slices == 1 or 2 * slices <= stages, what
            need = 4 * rows * N
            if layout == F.FL_GEMM_TN:
                rem = (M + 255) // 256 * (N // 256) % 256
                need = rem * 256 * 256 * 4
                assert slices == 1 or (tile == 256 and 0 < rem * slices <= 256), what
            assert slices == 1 or (slices * need <= part and tile != 192), what
            sliced += slices > 1
        if len(plan) == 2:
            assert layout != F.FL_GEMM_TN and plan[1][1] <= 128, what
            assert plan[0][0] % (256 if sums else plan[0][1]) == 0, what
            two += 1
    assert sliced > 100 and (two > 100 or layout == F.FL_GEMM_TN)
