"""GPU parity: the HIP path (through the C ABI) against the fp64 oracle, element by element."""
import numpy as np
import pytest

import paper_2602_24066_amd as S
from oracle import sig_oracle as O
from sig_workloads import (WORKLOADS, make_grad_coeffs, make_path, random_prefix_closed_words, workload_path)
from tests.gpu_common import (BWD_TOL, FWD_TOL, build_both, build_for_workload, check_parity, gpu_forward_backward,
                              oracle_backward, oracle_forward)

pytestmark = pytest.mark.gpu


# small cases: spans several work units, a ragged last group of paths (B not a multiple of 64),
# single-segment and single-path inputs
SMALL = [
    ("truncated", dict(d=2, depth=4), 32, 64, "iid"),
    ("truncated", dict(d=3, depth=5), 70, 33, "scaled"),
    ("truncated", dict(d=4, depth=6), 5, 17, "time0"),
    ("truncated", dict(d=8, depth=3), 129, 9, "iid"),
    ("truncated", dict(d=16, depth=3), 3, 40, "ar1"),
    ("truncated", dict(d=8, depth=5), 3, 21, "scaled"),
    ("truncated", dict(d=16, depth=4), 2, 19, "ar1"),
    # d = 1: a level is a single number (X_L - X_0)^n / n!; a path that returns towards its start cancels
    # it in fp32, so the one-letter case uses the monotone time channel (level n = 1/n!)
    ("truncated", dict(d=1, depth=6), 2, 12, "time0"),
    ("truncated", dict(d=5, depth=1), 65, 12, "iid"),
    ("truncated", dict(d=3, depth=4), 1, 1, "iid"),
    ("truncated", dict(d=2, depth=10), 4, 25, "iid"),
    ("anisotropic", dict(d=6, weights=(1, 1, 2, 2, 3, 3), cutoff=6.0), 66, 30, "iid"),
    # the only word of length 7 here is letter 0 seven times, (X_L - X_0)^7 / 7!: as for d = 1 the channel must
    # be monotone for that level to be well conditioned in fp32
    ("anisotropic", dict(d=3, weights=(1.0, 2.0, 1.5), cutoff=7.0), 10, 21, "time0"),
    ("words", dict(d=10, n_words=1500, max_len=6), 67, 20, "iid"),
    ("words", dict(d=4, n_words=400, max_len=9), 12, 15, "iid"),
    ("words", dict(d=40, n_words=300, max_len=3), 9, 10, "iid"),
]


@pytest.mark.parametrize("case", range(len(SMALL)))
def test_small_cases_elementwise(case):
    kind, kw, B, L, dist = SMALL[case]
    d = kw["d"]
    words = None
    if kind == "words":
        words = random_prefix_closed_words(100 + case, d, kw["n_words"], kw["max_len"])
    ws, W = build_both(kind, d, depth=kw.get("depth"), weights=kw.get("weights"), cutoff=kw.get("cutoff"), words=words)
    X = make_path(dist, 200 + case, B, L, d)
    G = make_grad_coeffs(300 + case, B, ws.size)
    check_parity(ws, W, kind, kw.get("depth"), X, G, what=f"small[{case}]")


def d4_inputs(seed, B, L):
    """Inputs for the register-resident d = 4 kernels: the monotone time channel of c2, and paths whose increments
    change sign in every channel (iid; per-channel scales for longer paths), so that chunk-boundary adjoints and the
    products in LDS see both signs everywhere."""
    dists = ["time0", "iid"] + (["scaled"] if L >= 64 else [])
    return [(dist, make_path(dist, seed + 7 * k, B, L, 4)) for k, dist in enumerate(dists)]


# Time chunks (Chen's relation between chunk signatures): forced chunk counts, including chunk lengths that do not
# divide L and a last chunk of a single segment; the automatic choice is exercised by the small batches below.
@pytest.mark.parametrize("d,depth,B,L,chunks", [(4, 6, 3, 97, 3), (4, 6, 2, 65, 2), (4, 6, 1, 160, 5), (8, 5, 2, 100, 3),
                                                (16, 4, 1, 129, 4), (4, 6, 2, 600, 0), (16, 4, 3, 700, 0)])
def test_time_chunks(monkeypatch, d, depth, B, L, chunks):
    if chunks:
        monkeypatch.setenv("SIG_CHUNKS", str(chunks))
    else:
        monkeypatch.delenv("SIG_CHUNKS", raising=False)
    ws, W = build_both("truncated", d, depth=depth)
    G = make_grad_coeffs(600 + L, B, ws.size)
    lib = S.load_library()
    if chunks:
        assert lib.sig_forward_workspace_bytes(ws._h, B, L + 1) >= 4 * B * chunks * ws.size
    else:
        assert lib.sig_forward_workspace_bytes(ws._h, B, L + 1) > 0      # few paths: chunking is chosen by itself
    inputs = d4_inputs(500 + L, B, L) if d == 4 else [("iid", make_path("iid", 500 + L, B, L, d))]
    for dist, X in inputs:
        check_parity(ws, W, "truncated", depth, X, G, what=f"chunks d={d} N={depth} L={L} C={chunks} {dist}")


# d = 4 backward with one wavefront per (path, chunk) row, forced for batches that would not select it
@pytest.mark.parametrize("B,L,chunks", [(3, 97, 3), (5, 17, 0), (130, 40, 0), (2, 160, 5), (1, 1, 0), (70, 64, 2)])
def test_backward_one_wavefront_per_row(monkeypatch, B, L, chunks):
    monkeypatch.setenv("SIG_BWD_TAILS", "1")
    if chunks:
        monkeypatch.setenv("SIG_CHUNKS", str(chunks))
    else:
        monkeypatch.delenv("SIG_CHUNKS", raising=False)
    ws, W = build_both("truncated", 4, depth=6)
    G = make_grad_coeffs(800 + L, B, ws.size)
    for dist, X in d4_inputs(700 + L, B, L):
        check_parity(ws, W, "truncated", 6, X, G, what=f"tails B={B} L={L} C={chunks} {dist}")


# ... and its fused form: the 2, 4 or 8 chunks of a path in one workgroup, chunk signatures and boundary adjoints in
# LDS; the last three cases take it by themselves (8, 4 and 2 chunks)
@pytest.mark.parametrize("B,L,chunks", [(3, 97, 4), (1, 33, 4), (5, 64, 4), (2, 35, 4), (1, 300, 4), (2, 2000, 4),
                                        (3, 17, 2), (70, 40, 2), (2, 16, 2), (2, 801, 2),
                                        (3, 97, 8), (1, 64, 8), (2, 67, 8), (5, 255, 8), (1, 1500, 8),
                                        (200, 100, 0), (300, 64, 0), (1000, 24, 0)])
def test_backward_chunks_in_one_workgroup(monkeypatch, B, L, chunks):
    if chunks:
        monkeypatch.setenv("SIG_BWD_TAILS", str(chunks))
    else:
        monkeypatch.delenv("SIG_BWD_TAILS", raising=False)
    monkeypatch.delenv("SIG_CHUNKS", raising=False)
    ws, W = build_both("truncated", 4, depth=6)
    G = make_grad_coeffs(950 + L, B, ws.size)
    lib = S.load_library()
    gdx = (4 * B * L * 4 + 255) // 256 * 256
    assert lib.sig_backward_workspace_bytes(ws._h, B, L + 1) == gdx       # no chunk arrays in device memory
    for dist, X in d4_inputs(900 + L, B, L):
        check_parity(ws, W, "truncated", 6, X, G, what=f"fused tails B={B} L={L} C={chunks} {dist}")


# forward with the 2 or 4 chunks of a path in one workgroup (d = 4, depth 6), forced for any batch size; the last
# two cases take it by themselves (batch sizes in its range)
@pytest.mark.parametrize("B,L,chunks", [(3, 97, 4), (1, 32, 4), (5, 64, 4), (2, 35, 4), (1, 300, 4), (3, 17, 2),
                                        (70, 40, 2), (2, 16, 2), (2, 1001, 2), (130, 50, 0), (400, 33, 0)])
def test_forward_chunks_in_one_workgroup(monkeypatch, B, L, chunks):
    if chunks:
        monkeypatch.setenv("SIG_FWD_TAILS", str(chunks))
    else:
        monkeypatch.delenv("SIG_FWD_TAILS", raising=False)
    monkeypatch.delenv("SIG_CHUNKS", raising=False)
    ws, W = build_both("truncated", 4, depth=6)
    assert ws.kernel_name(False, B, L + 1) == "trunc_tails_fwd_kernel"
    G = make_grad_coeffs(1350 + L, B, ws.size)
    for dist, X in d4_inputs(1300 + L, B, L):
        check_parity(ws, W, "truncated", 6, X, G, what=f"fused forward B={B} L={L} C={chunks} {dist}")


# Forward and backward with the time-chunk signatures kept between the two calls (checkpointed form): every chunk
# count, chunk lengths that do not divide L, the launcher's own choice, and shapes where it takes no chunks at all
@pytest.mark.parametrize("d,depth,B,L,chunks", [(8, 5, 2, 200, 0), (8, 5, 3, 131, 2), (8, 5, 2, 197, 3), (8, 5, 1, 260, 4),
                                                (16, 4, 2, 150, 2), (16, 4, 1, 200, 3), (16, 4, 2, 333, 0), (8, 5, 2, 40, 0),
                                                (16, 4, 1, 530, 0), (8, 5, 2, 600, 7), (8, 5, 40, 300, 0), (8, 5, 1, 1100, 0),
                                                (4, 6, 3, 300, 0),
                                                (3, 4, 5, 100, 0)])
def test_checkpointed_forward_and_backward(d, depth, B, L, chunks):
    import torch
    ws, W = build_both("truncated", d, depth=depth)
    if chunks:
        ws.set_option("ckpt_chunks", chunks)
    lib = S.load_library()
    nck = int(lib.sig_checkpoint_bytes(ws._h, B, L + 1))
    wanted = {8: 256, 16: 128}.get(d, 0)                  # rows that fill the chip with two wavefronts per SIMD
    expect_chunks = chunks if chunks else (min(16, -(-wanted // B), L // 64) if d in (8, 16) and L >= 128 else 0)
    if not chunks and expect_chunks > 4:
        expect_chunks = 16 if expect_chunks >= 16 else (8 if expect_chunks >= 8 else 4)    # beyond four: powers of two
    assert nck == (4 * B * expect_chunks * ws.size + 255) // 256 * 256
    X = make_path("iid", 2500 + L, B, L, d)
    G = make_grad_coeffs(2600 + L, B, ws.size)
    xp, grad = torch.from_numpy(X).cuda(), torch.from_numpy(G).cuda()
    coeffs, ck = S.sig_forward_checkpointed(ws, xp)
    assert ck.numel() == nck
    gp = S.sig_backward_checkpointed(ws, xp, coeffs, grad, ck)
    torch.cuda.synchronize()
    coeffs, gp = coeffs.cpu().numpy(), gp.cpu().numpy()
    lengths = np.array([len(w) for w in W])
    for n, e in O.level_errors(coeffs, O.forward_dense(X, depth), lengths).items():
        assert e <= FWD_TOL, f"checkpointed forward, level {n}: {e:.3e}"
    gerr = O.grad_errors(gp, O.backward_dense(X, depth, G.astype(np.float64)))
    assert gerr.max() <= BWD_TOL, f"checkpointed backward: {gerr.max():.3e}"


@pytest.mark.parametrize("d,depth,B,L,kept", [
    (8, 5, 5, 150, False),     # two chunks are kept, more are taken
    (16, 4, 2, 300, False),    # four and sixteen
    (8, 5, 20, 300, True),     # the four that are kept
    (16, 4, 12, 150, True),    # two; eight would be slower
])
def test_checkpointed_backward_with_the_stated_workspace(d, depth, B, L, kept):
    """With exactly the bytes it states the backward call takes the route its model chose: other chunks than are kept, seen by a
    checkpoint of NaN that it does not read, or the kept ones; the forward call of the pair needs no workspace at all."""
    import ctypes
    import torch
    ws, W = build_both("truncated", d, depth=depth)
    lib = S.load_library()
    X, G = make_path("iid", 2700 + L, B, L, d), make_grad_coeffs(2701, B, ws.size)
    x, g = torch.from_numpy(X).cuda(), torch.from_numpy(G).cuda()
    c = torch.empty((B, ws.size), device="cuda")
    ck = torch.empty(int(lib.sig_checkpoint_bytes(ws._h, B, L + 1)), dtype=torch.uint8, device="cuda")
    P = ctypes.c_void_p
    stream = P(torch.cuda.current_stream().cuda_stream)
    assert lib.sig_forward_checkpointed_workspace_bytes(ws._h, B, L + 1) == 0
    assert lib.sig_forward_checkpointed(ws._h, P(x.data_ptr()), B, L + 1, P(c.data_ptr()), P(ck.data_ptr()), ck.numel(), None, 0,
                                        stream) == 0
    n = int(lib.sig_backward_checkpointed_workspace_bytes(ws._h, B, L + 1))
    work = torch.empty(n, dtype=torch.uint8, device="cuda")
    gp = torch.empty_like(x)

    def call(bytes_):
        return lib.sig_backward_checkpointed(ws._h, P(x.data_ptr()), P(c.data_ptr()), P(g.data_ptr()), P(ck.data_ptr()), ck.numel(), B,
                                             L + 1, P(gp.data_ptr()), P(work.data_ptr()), bytes_, stream)

    if kept:
        assert call(n - 1) == -5
    assert call(n) == 0
    gref = oracle_backward(X, W, "truncated", depth, G.astype(np.float64))
    assert O.grad_errors(gp.cpu().numpy(), gref).max() <= BWD_TOL
    ck.view(torch.float32).fill_(float("nan"))
    assert call(n) == 0
    assert np.isnan(gp.cpu().numpy()).any() if kept else O.grad_errors(gp.cpu().numpy(), gref).max() <= BWD_TOL


@pytest.mark.parametrize("d,depth,B,L", [(8, 5, 3, 1100), (16, 4, 2, 1030)])
def test_long_paths_need_the_short_rows_of_their_chunks_alone(d, depth, B, L):
    """sig_forward takes one array of chunk signatures, sig_backward the gradient of the increments and rows of the words shorter
    than the depth: those bytes are accepted, also where a caller is told the size of whole arrays, and fewer are refused."""
    import ctypes
    import torch
    ws, W = build_both("truncated", d, depth=depth)
    lib = S.load_library()
    X, G = make_path("iid", 2800 + L, B, L, d), make_grad_coeffs(2801, B, ws.size)
    x, g = torch.from_numpy(X).cuda(), torch.from_numpy(G).cuda()
    c, gp = torch.empty((B, ws.size), device="cuda"), torch.empty_like(x)
    gdx, low = (4 * B * L * d + 255) // 256 * 256, int(ws.level_start[depth])
    array = (4 * B * 4 * ws.size + 255) // 256 * 256                 # four chunks of 256 segments
    rows = 3 * ((4 * B * 16 * low + 255) // 256 * 256) + (4 * B * 15 * low + 255) // 256 * 256      # sixteen chunks
    work = torch.empty(array + gdx + rows, dtype=torch.uint8, device="cuda")
    P = ctypes.c_void_p
    stream = P(torch.cuda.current_stream().cuda_stream)

    def forward(n):
        return lib.sig_forward(ws._h, P(x.data_ptr()), B, L + 1, P(c.data_ptr()), P(work.data_ptr()), n, stream)

    def backward(n):
        return lib.sig_backward(ws._h, P(x.data_ptr()), P(c.data_ptr()), P(g.data_ptr()), B, L + 1, P(gp.data_ptr()), P(work.data_ptr()),
                                n, stream)

    assert forward(array - 1) == -5 and forward(array) == 0
    assert backward(gdx) == -5 and backward(gdx + rows) == 0
    assert gdx + rows < lib.sig_backward_workspace_bytes(ws._h, B, L + 1)
    lengths = np.array([len(w) for w in W])
    O.set_threads(2)
    try:
        errs = O.level_errors(c.cpu().numpy(), oracle_forward(X, W, "truncated", depth), lengths)
        gref = oracle_backward(X, W, "truncated", depth, G.astype(np.float64))
    finally:
        O.set_threads(16)
    assert max(errs.values()) <= FWD_TOL, errs
    assert O.grad_errors(gp.cpu().numpy(), gref).max() <= BWD_TOL


def _no_repeat_words(d, n):
    """Words of up to n letters in which no letter follows itself: closed under prefixes and suffixes."""
    out, level = [], [(i,) for i in range(d)]
    for _ in range(n):
        out += level
        level = [w + (i,) for w in level for i in range(d) if i != w[-1]]
    return out


# The same pair of calls on word sets closed under suffixes (anisotropic sets; a word list that is): chunk counts by the
# library's rule (two and eight) and forced (two, three, four), chunk lengths that do not divide L, a batch of more than one lane group, against the
# oracle; and a list that lacks suffixes, which takes no chunks.  (Every length of these sets has several words: a length
# with a single word is ill-conditioned under the forward error measure for any summation order.)
WORD_CHUNK_CASES = {
    "aniso3": ("anisotropic", 3, (1.0, 1.25, 1.5), 4.5, None, 5, 200, 3, 3),
    "aniso6": ("anisotropic", 6, (1, 1, 2, 2, 3, 3), 8.0, None, 70, 257, 0, 2),
    "aniso6-forced": ("anisotropic", 6, (1, 1, 2, 2, 3, 3), 8.0, None, 70, 257, 4, 4),
    "aniso3-rule": ("anisotropic", 3, (1.0, 1.25, 1.5), 4.5, None, 2, 1030, 0, 8),
    "aniso2-forced": ("anisotropic", 2, (0.3, 0.4), 1.6, None, 3, 300, 2, 2),
    "no-repeat": ("list", 3, None, None, "no-repeat", 9, 130, 2, 2),
    "random": ("list", 4, None, None, "random", 4, 200, 0, 0),
}


@pytest.mark.parametrize("case", list(WORD_CHUNK_CASES))
def test_checkpointed_word_sets(case):
    import torch
    kind, d, weights, cutoff, which, B, L, forced, expect_chunks = WORD_CHUNK_CASES[case]
    words = None
    if which == "no-repeat":
        words = _no_repeat_words(d, 5)
    elif which == "random":
        words = random_prefix_closed_words(11, d, 80, 5)
    ws, W = build_both(kind, d, weights=weights, cutoff=cutoff, words=words)
    if forced:
        ws.set_option("ckpt_chunks", forced)
    assert ws.suffix_closed == (which != "random")
    lib = S.load_library()
    nck = int(lib.sig_checkpoint_bytes(ws._h, B, L + 1))
    assert nck == (4 * B * expect_chunks * ws.size + 255) // 256 * 256
    X = make_path("iid", 5100 + L, B, L, d)
    G = make_grad_coeffs(5200 + L, B, ws.size)
    xp, grad = torch.from_numpy(X).cuda(), torch.from_numpy(G).cuda()
    coeffs, ck = S.sig_forward_checkpointed(ws, xp)
    gp = S.sig_backward_checkpointed(ws, xp, coeffs, grad, ck)
    plain = S.sig_forward(ws, xp)
    gplain = S.sig_backward(ws, xp, plain, grad)
    torch.cuda.synchronize()
    if expect_chunks:                      # the checkpoint holds the signatures of the chunks: the first is that of the first Lc segments
        Lc = -(-L // expect_chunks)
        first = ck.view(torch.float32)[: B * expect_chunks * ws.size].view(B, expect_chunks, ws.size)[:, 0].cpu().numpy()
        ref_first = O.forward_words(np.ascontiguousarray(X[:, : Lc + 1]), W)
        for n, e in O.level_errors(first, ref_first, np.array([len(w) for w in W])).items():
            assert e <= FWD_TOL, f"{case}: first chunk signature, level {n}: {e:.3e}"
    coeffs, gp = coeffs.cpu().numpy(), gp.cpu().numpy()
    lengths = np.array([len(w) for w in W])
    ref = O.forward_words(X, W)
    for n, e in O.level_errors(coeffs, ref, lengths).items():
        assert e <= FWD_TOL, f"{case}: checkpointed forward, level {n}: {e:.3e}"
    gref = O.backward_words(X, W, G.astype(np.float64))
    gerr = O.grad_errors(gp, gref)
    assert gerr.max() <= BWD_TOL, f"{case}: checkpointed backward: {gerr.max():.3e}"
    assert O.grad_errors(gplain.cpu().numpy(), gref).max() <= BWD_TOL
    # sig_forward takes the same chunks, with the chunk signatures in its workspace
    for n, e in O.level_errors(plain.cpu().numpy(), ref, lengths).items():
        assert e <= FWD_TOL, f"{case}: sig_forward, level {n}: {e:.3e}"


@pytest.mark.parametrize("d,depth,B,L", [(8, 5, 3, 1100), (16, 4, 2, 1030)])
def test_plain_backward_takes_time_chunks_for_few_long_paths(d, depth, B, L):
    """sig_backward on few long paths of a full truncation recomputes the chunk signatures and walks chunks side by side (the
    stated size of its workspace is that of four arrays of four whole chunk signatures; the call takes less, short rows of
    more chunks); the result is the oracle's, and that of the entry point with the static scratch array, which always
    walks whole paths."""
    import torch
    ws, W = build_both("truncated", d, depth=depth)
    lib = S.load_library()
    gdx = (4 * B * L * d + 255) // 256 * 256
    per_array = (4 * B * 4 * ws.size + 255) // 256 * 256
    assert lib.sig_backward_workspace_bytes(ws._h, B, L + 1) == gdx + 4 * per_array
    X = make_path("iid", 6100 + L, B, L, d)
    G = make_grad_coeffs(6200 + L, B, ws.size)
    xp, grad = torch.from_numpy(X).cuda(), torch.from_numpy(G).cuda()
    coeffs = S.sig_forward(ws, xp)
    gp = S.sig_backward(ws, xp, coeffs, grad)
    gs = torch.empty_like(xp)
    S.sig_backward_static(ws, xp, coeffs, grad, gs)
    torch.cuda.synchronize()
    O.set_threads(2)
    try:
        gref = O.backward_dense(X, depth, G.astype(np.float64))
    finally:
        O.set_threads(16)
    assert O.grad_errors(gp.cpu().numpy(), gref).max() <= BWD_TOL
    assert O.grad_errors(gs.cpu().numpy(), gref).max() <= BWD_TOL


@pytest.mark.parametrize("kind,d,n_words,max_len,B,L,chunks", [
    ("words", 4, 60, 4, 3, 50, 3),         # closure of 78 words: one word a thread, three terms
    ("words", 10, 700, 6, 2, 37, 2),       # 1,907 words: two a thread, five terms; the last chunk shorter
    ("words", 6, 1200, 8, 65, 33, 5),      # 3,801 words: four a thread, seven terms; two path groups
    ("words", 5, 300, 5, 70, 200, 0),      # the library's own count
    ("leadlag", 2, None, 3, 39, 150, 16),  # 36 words, closure of 38
    ("aniso", 3, None, None, 4, 90, 6),    # closed under suffixes itself
    ("letters", 3, None, 1, 5, 24, 4),     # words of one letter: no terms
])
def test_time_chunks_of_small_launches(kind, d, n_words, max_len, B, L, chunks):
    """sig_forward and sig_backward cut the paths of small launches into time chunks, also for sets that lack suffixes (through
    their closure): both against the oracle, and the entry point that walks whole paths after them."""
    import torch
    if kind == "aniso":
        ws, W = build_both("anisotropic", d, weights=(1.0, 1.25, 1.5), cutoff=4.5)
    elif kind == "leadlag":
        ws = S.sig_wordset_build_leadlag_sparse(d, max_len)
        ws.upload("cuda:0")
        W, d = O.prefix_closure(O.leadlag_sparse_words(d, max_len)), 2 * d
    else:
        words = [(i,) for i in range(d)] if kind == "letters" else random_prefix_closed_words(41, d, n_words, max_len)
        ws, W = build_both("words", d, words=words)
    lib = S.load_library()
    whole = int(lib.sig_backward_workspace_bytes(ws._h, B, 8))
    ws.set_option("chunks", chunks)
    assert int(lib.sig_backward_workspace_bytes(ws._h, B, L + 1)) > whole and int(lib.sig_forward_workspace_bytes(ws._h, B, L + 1)) > 0
    X = make_path("iid", 7100 + L, B, L, d)
    G = make_grad_coeffs(7200 + L, B, ws.size)
    xp, grad = torch.from_numpy(X).cuda(), torch.from_numpy(G).cuda()
    coeffs = S.sig_forward(ws, xp)
    gp = S.sig_backward(ws, xp, coeffs, grad)
    gs = torch.empty_like(xp)
    S.sig_backward_static(ws, xp, coeffs, grad, gs)
    torch.cuda.synchronize()
    lengths = np.array([len(w) for w in W])
    for n, e in O.level_errors(coeffs.cpu().numpy(), O.forward_words(X, W), lengths).items():
        assert e <= FWD_TOL, f"level {n}: {e:.3e}"
    gref = O.backward_words(X, W, G.astype(np.float64))
    assert O.grad_errors(gp.cpu().numpy(), gref).max() <= BWD_TOL
    assert O.grad_errors(gs.cpu().numpy(), gref).max() <= BWD_TOL


def test_time_chunks_of_small_launches_under_capture():
    """What a call under graph capture may not load it does without: after one eager step on short paths a step on long ones is
    recorded with whole paths, and after one on long paths a step on short ones as well."""
    import torch
    words = random_prefix_closed_words(43, 5, 120, 5)
    for eager, captured in ((12, 160), (160, 12)):
        ws, W = build_both("words", 5, words=words)
        B = 6
        X = [make_path("iid", 7300 + n, B, n, 5) for n in (eager, captured)]
        xs = [torch.from_numpy(x).cuda() for x in X]
        G = make_grad_coeffs(7301, B, ws.size)
        g = torch.from_numpy(G).cuda()
        S.sig_backward(ws, xs[0], S.sig_forward(ws, xs[0]), g)
        lib = S.load_library()
        wf = torch.empty(max(int(lib.sig_forward_workspace_bytes(ws._h, B, captured + 1)), 256), dtype=torch.uint8, device="cuda")
        wb = torch.empty(int(lib.sig_backward_workspace_bytes(ws._h, B, captured + 1)), dtype=torch.uint8, device="cuda")
        c, gp = torch.zeros((B, ws.size), device="cuda"), torch.zeros_like(xs[1])
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            S.sig_forward(ws, xs[1], out=c, workspace=wf)
            S.sig_backward(ws, xs[1], c, g, out=gp, workspace=wb)
        gref = O.backward_words(X[1], W, G.astype(np.float64))
        for rep in range(3):
            xs[1].copy_(torch.from_numpy(X[1]))
            gp.fill_(5.0)
            graph.replay()
            torch.cuda.synchronize()
            for n, e in O.level_errors(c.cpu().numpy(), O.forward_words(X[1], W), np.array([len(w) for w in W])).items():
                assert e <= FWD_TOL, (rep, n, e)
            assert O.grad_errors(gp.cpu().numpy(), gref).max() <= BWD_TOL, rep
            S.sig_forward(ws, xs[0])


@pytest.mark.parametrize("d,depth,B,L,chunks", [
    (8, 5, 2, 70, 2), (8, 5, 3, 50, 5), (8, 5, 1, 200, 0), (8, 5, 70, 40, 3), (16, 4, 2, 70, 3), (16, 4, 1, 33, 8),
    (16, 4, 3, 150, 0), (16, 4, 30, 40, 4)])
def test_time_chunks_of_truncations_by_slices(d, depth, B, L, chunks):
    """Few paths of the precompiled truncations with 8 and 16 letters: chunk products by slices in both directions (chunks that do
    not divide the length, one to 16 of them, rows for one and for two wavefronts per SIMD), and the walk over whole paths that a
    caller with the workspace for that gets."""
    import ctypes
    import torch
    ws, _ = build_both("truncated", d, depth=depth)
    lib = S.load_library()
    X = make_path("iid", 7400 + L, B, L, d)
    G = make_grad_coeffs(7500 + L, B, ws.size)
    xp, grad = torch.from_numpy(X).cuda(), torch.from_numpy(G).cuda()
    if chunks:
        ws.set_option("chunks", chunks)
    gdx = (4 * B * L * d + 255) // 256 * 256
    nf, nb = int(lib.sig_forward_workspace_bytes(ws._h, B, L + 1)), int(lib.sig_backward_workspace_bytes(ws._h, B, L + 1))
    assert nf > 0 and nb > gdx
    coeffs = S.sig_forward(ws, xp)
    gp = S.sig_backward(ws, xp, coeffs, grad)
    c2, g2 = torch.empty_like(coeffs), torch.empty_like(xp)
    P = ctypes.c_void_p
    wk = torch.empty(nb, dtype=torch.uint8, device="cuda")
    ws.set_option("chunks", 0)
    stream = P(torch.cuda.current_stream().cuda_stream)
    assert lib.sig_forward(ws._h, P(xp.data_ptr()), B, L + 1, P(c2.data_ptr()), None, 0, stream) == 0
    assert lib.sig_backward(ws._h, P(xp.data_ptr()), P(coeffs.data_ptr()), P(grad.data_ptr()), B, L + 1, P(g2.data_ptr()),
                            P(wk.data_ptr()), gdx, stream) == 0
    torch.cuda.synchronize()
    lengths = np.array([len(w) for w in O.truncated_words(d, depth)])
    ref, gref = O.forward_dense(X, depth), O.backward_dense(X, depth, G.astype(np.float64))
    for c, g in ((coeffs, gp), (c2, g2)):
        for n, e in O.level_errors(c.cpu().numpy(), ref, lengths).items():
            assert e <= FWD_TOL, f"level {n}: {e:.3e}"
        assert O.grad_errors(g.cpu().numpy(), gref).max() <= BWD_TOL


def test_checkpointed_word_sets_reject_bad_buffers():
    """Buffers that are missing, too small or misaligned are refused with an error code before anything is launched."""
    import ctypes
    import torch
    ws, W = build_both("anisotropic", 3, weights=(1.0, 1.25, 1.5), cutoff=4.5)
    ws.set_option("ckpt_chunks", 3)
    lib = S.load_library()
    B, L = 5, 200
    nck = int(lib.sig_checkpoint_bytes(ws._h, B, L + 1))
    nf = int(lib.sig_forward_checkpointed_workspace_bytes(ws._h, B, L + 1))
    nb = int(lib.sig_backward_checkpointed_workspace_bytes(ws._h, B, L + 1))
    assert nck > 0 and nf > 0 and nb > 0
    xp = torch.from_numpy(make_path("iid", 5300, B, L, 3)).cuda()
    grad = torch.from_numpy(make_grad_coeffs(5301, B, ws.size)).cuda()
    coeffs = torch.full((B, ws.size), 3.0, dtype=torch.float32, device="cuda")
    gpath = torch.full((B, L + 1, 3), 3.0, dtype=torch.float32, device="cuda")
    ck = torch.zeros(nck + 256, dtype=torch.uint8, device="cuda")
    wk = torch.zeros(max(nf, nb) + 256, dtype=torch.uint8, device="cuda")
    assert ck.data_ptr() % 256 == 0 and wk.data_ptr() % 256 == 0
    P = ctypes.c_void_p

    def fwd(ckp, ckn, wp, wn):
        return lib.sig_forward_checkpointed(ws._h, P(xp.data_ptr()), B, L + 1, P(coeffs.data_ptr()), P(ckp), ckn, P(wp), wn, None)

    def bwd(ckp, ckn, wp, wn):
        return lib.sig_backward_checkpointed(ws._h, P(xp.data_ptr()), P(coeffs.data_ptr()), P(grad.data_ptr()), P(ckp), ckn, B, L + 1,
                                             P(gpath.data_ptr()), P(wp), wn, None)

    for call, need in ((fwd, nf), (bwd, nb)):
        assert call(ck.data_ptr(), nck - 1, wk.data_ptr(), need) == -5
        assert call(0, nck, wk.data_ptr(), need) == -5
        assert call(ck.data_ptr(), nck, wk.data_ptr(), need - 1) == -5
        assert call(ck.data_ptr(), nck, 0, need) == -5
        assert call(ck.data_ptr() + 4, nck, wk.data_ptr(), need) == -1
        assert call(ck.data_ptr(), nck, wk.data_ptr() + 4, need) == -1
    torch.cuda.synchronize()
    assert (coeffs == 3.0).all() and (gpath == 3.0).all() and (ck == 0).all()      # nothing ran
    assert fwd(ck.data_ptr(), nck, wk.data_ptr(), nf) == 0 and bwd(ck.data_ptr(), nck, wk.data_ptr(), nb) == 0
    torch.cuda.synchronize()
    gref = O.backward_words(xp.cpu().numpy(), W, grad.cpu().numpy().astype(np.float64))
    assert O.grad_errors(gpath.cpu().numpy(), gref).max() <= BWD_TOL


# Every tile shape of the d = 16 and d = 8 backward kernels, forced on batches far too small to take them by themselves:
# tiles that do not divide the number of segments, a single ragged tile, with and without time chunks
@pytest.mark.parametrize("d,depth,tile", [(16, 4, 4), (16, 4, 8), (16, 4, 12), (16, 4, 16), (8, 5, 4), (8, 5, 8), (8, 5, 16)])
@pytest.mark.parametrize("B,L,chunks", [(2, 77, 0), (1, 9, 0), (3, 150, 2)])
def test_backward_tile_shapes(d, depth, tile, B, L, chunks):
    import torch
    ws, W = build_both("truncated", d, depth=depth)
    ws.set_option("bwd_tile", tile)
    X = make_path("iid", 2900 + L + tile, B, L, d)
    G = make_grad_coeffs(3000 + L + tile, B, ws.size)
    gref = O.backward_dense(X, depth, G.astype(np.float64))
    xp, grad = torch.from_numpy(X).cuda(), torch.from_numpy(G).cuda()
    if chunks:
        ws.set_option("ckpt_chunks", chunks)
        coeffs, ck = S.sig_forward_checkpointed(ws, xp)
        gp = S.sig_backward_checkpointed(ws, xp, coeffs, grad, ck)
    else:
        coeffs = S.sig_forward(ws, xp)
        gp = S.sig_backward(ws, xp, coeffs, grad)
    torch.cuda.synchronize()
    gerr = O.grad_errors(gp.cpu().numpy(), gref)
    assert gerr.max() <= BWD_TOL, f"d={d} tile={tile} B={B} L={L} chunks={chunks}: {gerr.max():.3e}"


@pytest.mark.parametrize("d,depth,B,L", [(8, 5, 2, 300), (16, 4, 2, 400), (4, 6, 3, 257)])
def test_reconstruction_returns_to_the_empty_signature(d, depth, B, L):
    """Stepping the terminal signature back through all segments (Proposition 4.6) must end at the signature of the
    empty path (Lemma 4.5): the kernels report the largest coefficient they are left with, and the gradient of the
    same call is the ordinary one."""
    import torch
    ws, W = build_both("truncated", d, depth=depth)
    X = make_path("iid", 2700 + L, B, L, d)
    G = make_grad_coeffs(2800 + L, B, ws.size)
    xp, grad = torch.from_numpy(X).cuda(), torch.from_numpy(G).cuda()
    coeffs = S.sig_forward(ws, xp)
    gp, resid = S.sig_backward_residual(ws, xp, coeffs, grad)
    torch.cuda.synchronize()
    resid = resid.cpu().numpy()
    scale = float(coeffs.abs().max())
    assert resid.shape == (B,) and np.all(resid >= 0.0) and resid.max() <= 1e-4 * max(scale, 1.0), (resid, scale)
    gerr = O.grad_errors(gp.cpu().numpy(), O.backward_dense(X, depth, G.astype(np.float64)))
    assert gerr.max() <= BWD_TOL
    # a terminal signature that is not the path's own does not come back to zero: the check discriminates
    wrong = coeffs.clone()
    wrong[:, 0] += 0.5
    _, resid2 = S.sig_backward_residual(ws, xp, wrong, grad)
    assert float(resid2.min()) > 0.1


@pytest.mark.parametrize("d,depth,B,L", [(8, 5, 2, 70), (16, 4, 1, 300), (4, 6, 3, 40), (8, 5, 2, 1100)])
def test_residual_needs_the_workspace_of_whole_paths_alone(d, depth, B, L):
    """sig_backward_residual walks whole paths: the gradient of the increments is all that its workspace has to hold, also where
    sig_backward takes time chunks; a byte less is refused."""
    import ctypes
    import torch
    ws, W = build_both("truncated", d, depth=depth)
    lib = S.load_library()
    gdx = (4 * B * L * d + 255) // 256 * 256
    X, G = make_path("iid", 7600 + L, B, L, d), make_grad_coeffs(7601, B, ws.size)
    x, g = torch.from_numpy(X).cuda(), torch.from_numpy(G).cuda()
    c = S.sig_forward(ws, x)
    gp, res = torch.full_like(x, float("nan")), torch.full((B,), float("nan"), device="cuda")
    work = torch.empty(gdx, dtype=torch.uint8, device="cuda")
    P = ctypes.c_void_p

    def call(n):
        return lib.sig_backward_residual(ws._h, P(x.data_ptr()), P(c.data_ptr()), P(g.data_ptr()), B, L + 1, P(gp.data_ptr()),
                                         P(res.data_ptr()), P(work.data_ptr()), n, P(torch.cuda.current_stream().cuda_stream))

    assert call(gdx - 1) == -5 and call(gdx) == 0
    torch.cuda.synchronize()
    assert float(res.max()) <= 1e-3
    assert O.grad_errors(gp.cpu().numpy(), oracle_backward(X, W, "truncated", depth, G.astype(np.float64))).max() <= BWD_TOL


def test_forward_fused_and_four_wavefront_kernels_agree():
    ws, W = build_both("truncated", 4, depth=6)
    X = make_path("time0", 21, 200, 255, 4)
    G = make_grad_coeffs(22, 200, ws.size)
    ws.set_option("fwd_tails", 0)
    assert ws.kernel_name(False, 200, 256) == "trunc_mfma_fwd_kernel"
    c0, _ = gpu_forward_backward(ws, X, G)
    ws.set_option("fwd_tails", -1)
    assert ws.kernel_name(False, 200, 256) == "trunc_tails_fwd_kernel"
    c4, _ = gpu_forward_backward(ws, X, G)
    lengths = np.array([len(w) for w in W])
    for n, e in O.level_errors(c4, c0.astype(np.float64), lengths).items():
        assert e <= 1e-5, (n, e)


@pytest.mark.parametrize("chunks", [2, 4, 8])
@pytest.mark.parametrize("L", [16, 17, 33, 64, 71, 155])
def test_chunks_of_the_fused_backward(chunks, L):
    """Every chunk's lanes work out the signature and the adjoints at its end; chunks of whole tiles, of a part of one, and shorter
    last ones."""
    ws, W = build_both("truncated", 4, depth=6)
    ws.set_option("bwd_tails", chunks)
    X = make_path("iid", 50 + L, 3, L, 4)
    G = make_grad_coeffs(60 + L, 3, ws.size)
    _, gp = gpu_forward_backward(ws, X, G)
    assert O.grad_errors(gp, oracle_backward(X, W, "truncated", 6, G.astype(np.float64))).max() <= BWD_TOL


@pytest.mark.parametrize("d,depth,B,Ls", [(4, 6, 3, (1, 7, 8, 9, 33)), (8, 5, 2, (1, 2, 7, 8, 9, 16, 17)), (16, 4, 2, (1, 15, 16, 17, 22)),
                                          (16, 4, 70, (21, 33))])
def test_partial_tiles_of_the_truncation_kernels(d, depth, B, Ls):
    """The kernels stop at a row's last segment instead of walking its last tile to the end: lengths around whole tiles, with LDS
    that the length before has filled."""
    ws, W = build_both("truncated", d, depth=depth)
    lengths = np.array([len(w) for w in W])
    for L in Ls:
        X = make_path("iid", 80 + L, B, L, d)
        G = make_grad_coeffs(90 + L, B, ws.size)
        c, gp = gpu_forward_backward(ws, X, G)
        few = min(B, 3)
        errs = O.level_errors(c[:few], oracle_forward(X[:few], W, "truncated", depth), lengths)
        assert max(errs.values()) <= FWD_TOL, (L, errs)
        gref = oracle_backward(X[:few], W, "truncated", depth, G[:few].astype(np.float64))
        assert O.grad_errors(gp[:few], gref).max() <= BWD_TOL, L


def test_rows_that_are_not_16_byte_aligned():
    """coeffs / grad_coeffs four bytes off a 16-byte boundary: the d = 4 kernels that use vector loads and stores step
    aside for the ones that do not, with the same results."""
    import torch
    ws, W = build_both("truncated", 4, depth=6)
    B, L = 130, 70
    X = make_path("time0", 31, B, L, 4)
    G = make_grad_coeffs(32, B, ws.size)
    xp = torch.from_numpy(X).cuda()
    buf_c = torch.empty(B * ws.size + 1, dtype=torch.float32, device="cuda")
    buf_g = torch.empty(B * ws.size + 1, dtype=torch.float32, device="cuda")
    c_off = buf_c[1:].view(B, ws.size)
    g_off = buf_g[1:].view(B, ws.size)
    assert c_off.data_ptr() % 16 == 4 and c_off.is_contiguous()
    g_off.copy_(torch.from_numpy(G))
    S.sig_forward(ws, xp, out=c_off)
    gp_off = S.sig_backward(ws, xp, c_off, g_off)
    c = S.sig_forward(ws, xp)
    gp = S.sig_backward(ws, xp, c, torch.from_numpy(G).cuda())
    lengths = np.array([len(w) for w in W])
    for n, e in O.level_errors(c_off.cpu().numpy(), c.cpu().numpy().astype(np.float64), lengths).items():
        assert e <= 1e-5, (n, e)
    assert O.grad_errors(gp_off.cpu().numpy(), gp.cpu().numpy().astype(np.float64)).max() <= 1e-4
    for n, e in O.level_errors(c_off.cpu().numpy(), O.forward_words(X, W), lengths).items():
        assert e <= FWD_TOL, (n, e)
    assert O.grad_errors(gp_off.cpu().numpy(), O.backward_words(X, W, G.astype(np.float64))).max() <= BWD_TOL


def test_chunked_and_unchunked_agree():
    ws, W = build_both("truncated", 4, depth=6)
    X = make_path("iid", 11, 4, 128, 4)
    G = make_grad_coeffs(12, 4, ws.size)
    ws.set_option("chunks", 1)
    c1, g1 = gpu_forward_backward(ws, X, G)
    ws.set_option("chunks", 4)
    c4, g4 = gpu_forward_backward(ws, X, G)
    lengths = np.array([len(w) for w in W])
    for n, e in O.level_errors(c4, c1.astype(np.float64), lengths).items():
        assert e <= 1e-5, (n, e)
    assert O.grad_errors(g4, g1.astype(np.float64)).max() <= 1e-4


@pytest.mark.parametrize("kind", ["anisotropic", "words"])
def test_table_driven_kernels(monkeypatch, kind):
    """With run-time specialisation switched off the table-driven kernels serve the same word sets."""
    monkeypatch.setenv("SIG_NO_JIT", "1")
    if kind == "anisotropic":
        ws, W = build_both(kind, 4, weights=(1.0, 1.0, 2.0, 3.0), cutoff=5.0)
    else:
        ws, W = build_both(kind, 6, words=random_prefix_closed_words(77, 6, 800, 5))
    assert ws.kernel_name(False) == "fwd_generic_kernel" and ws.kernel_name(True) == "bwd_generic_kernel"
    X = make_path("iid", 78, 70, 19, ws.dim)
    G = make_grad_coeffs(79, 70, ws.size)
    check_parity(ws, W, kind, None, X, G, what=f"table-driven {kind}")


@pytest.mark.parametrize("B,L", [(1000, 9), (1024, 16)])
def test_specialised_backward_with_intermediates_of_its_own(B, L):
    """Short units of two wavefronts a SIMD reconstruct from a second set of intermediates; a ragged group and tile among them."""
    ws, W = build_both("words", 6, words=random_prefix_closed_words(78, 6, 740, 6))
    ws.set_option("jit_waves", 2048)
    ws.set_option("chunks", 1)
    assert "const float m1_1 = " in ws.jit_source(True, B)
    X = make_path("iid", 81, B, L, 6)
    G = make_grad_coeffs(82, B, ws.size)
    check_parity(ws, W, "words", None, X, G, sample=[0, 1, 63, 64, 959, 960, B - 1], what=f"own set {B} x {L}")


def test_many_short_paths():
    """More paths than the register-resident kernels take in one launch (65,535): the specialised kernels serve a
    full truncation too.  Sampled paths against the oracle."""
    ws, W = build_both("truncated", 4, depth=6)
    B, L = 66000, 3
    X = make_path("iid", 41, B, L, 4)
    G = make_grad_coeffs(42, B, ws.size)
    sample = [0, 1, 63, 64, 4095, 65535, 65536, B - 1]
    check_parity(ws, W, "truncated", 6, X, G, sample=sample, what="B=66000")


@pytest.mark.parametrize("d,depth,B", [(8, 5, 60000), (4, 6, 400000)])
def test_more_than_2_to_the_31_coefficients(d, depth, B):
    """Row offsets in 64 bits: 60,000 paths of the (8, 5) truncation are 2.25e9 coefficients (9 GB per array), and so
    are 400,000 paths of the (4, 6) truncation, which the run-time specialised kernels serve (lanes = paths).
    Sampled paths against the oracle, among them the row in which the element index passes 2^31 and the last one.
    The cotangent is drawn on the device (a seeded input; 2e9 normals would take the host half a minute)."""
    import torch
    ws, W = build_both("truncated", d, depth=depth)
    L = 2
    assert B * ws.size > 2**31
    X = make_path("iid", 43, B, L, d)
    xp = torch.from_numpy(X).cuda()
    gen = torch.Generator(device="cuda").manual_seed(44)
    G = torch.randn((B, ws.size), device="cuda", dtype=torch.float32, generator=gen)
    coeffs = S.sig_forward(ws, xp)
    gp = S.sig_backward(ws, xp, coeffs, G)
    torch.cuda.synchronize()
    edge = 2**31 // ws.size
    idx = np.array([0, 1, 4095, edge - 1, edge, edge + 1, B - 2, B - 1])
    sel = torch.from_numpy(idx).cuda()
    c, g, gg = coeffs[sel].cpu().numpy(), gp[sel].cpu().numpy(), G[sel].cpu().numpy()
    del coeffs, G
    Xs = np.ascontiguousarray(X[idx])
    lengths = np.array([len(w) for w in W])
    for n, e in O.level_errors(c, O.forward_dense(Xs, depth), lengths).items():
        assert e <= FWD_TOL, (n, e)
    gerr = O.grad_errors(g, O.backward_dense(Xs, depth, gg.astype(np.float64)))
    assert gerr.max() <= BWD_TOL, gerr
    assert torch.isfinite(gp).all()


@pytest.mark.parametrize("d,depth,B,L,levels", [
    (6, 5, 3, 21, 2),     # two levels per lane, 216 words of length 3: three full wavefronts and a ragged one
    (6, 5, 2, 13, 1),     # one level per lane: 1,296 lanes; the first chain letter runs over 216 of them
    (3, 6, 5, 33, 2),     # 81 lanes per path
    (3, 6, 2, 20, 1),     # 243 lanes
    (2, 7, 4, 9, 2),      # half a wavefront per path
    (7, 4, 2, 17, 2),     # 49 lanes
    (7, 4, 2, 17, 1),     # 343 lanes
    (5, 3, 6, 8, 2),      # 5 lanes per path (forced: the launcher would take lanes = paths)
    (10, 4, 2, 19, 2),    # 100 lanes with 110 coefficients each, tiles of 6 segments
    (10, 4, 1, 25, 1),    # 1,000 lanes
    (9, 4, 3, 1, 1),      # a single segment
    (12, 3, 2, 11, 1),    # 144 lanes, tiles of 5 segments
    (12, 4, 1, 7, 1),     # the first chain letter changes inside some wavefronts (runs of 144 lanes)
    (6, 6, 1, 6, 2),      # runs of 216, 36, 6 and 1 lanes
    (3, 8, 2, 10, 2),     # six chain letters, two of them with runs of 64 lanes or more
    (40, 3, 1, 5, 1),     # tiles of one segment, 65,640 coefficients from a single path
])
def test_truncations_with_lanes_as_words(d, depth, B, L, levels, monkeypatch):
    """Full truncations that have no register-resident kernel of their own: the run-time compiled kernels with a
    word per lane, in both of their forms (the d leaves, or the d children and d^2 leaves, below the lane's word),
    every coefficient and the whole gradient against the oracle."""
    monkeypatch.setenv("SIG_LANES", "1")
    monkeypatch.setenv("SIG_LANES_LEVELS", str(levels))
    ws, W = build_both("truncated", d, depth=depth)
    assert ws.kernel_name(False, B, L + 1) == "sig_fwd_lanes" and ws.kernel_name(True, B, L + 1) == "sig_bwd_lanes"
    assert f"#define R {levels}\n" in ws.jit_source(False, B) and f"#define R {levels}\n" in ws.jit_source(True, B)
    X = make_path("iid", 71 + d, B, L, d)
    G = make_grad_coeffs(72 + d, B, ws.size)
    check_parity(ws, W, "truncated", depth, X, G, what=f"lanes = words, d={d} N={depth}, {levels} levels per lane")


@pytest.mark.parametrize("depth,B,L,levels,msum", [
    (7, 1024, 11, 0, 1),     # one wavefront per SIMD: matrix products
    (7, 1025, 11, 0, 0),     # more: sums by rows
    (8, 1300, 9, 0, 0),      # two levels per lane, a chain of six
    (9, 520, 19, 0, 0),      # chains of seven and of ten: one segment after the other, three long runs
    (12, 64, 5, 0, 0),
    (8, 1030, 17, 1, 0),     # one level, a chain of seven
])
def test_two_letters_with_many_paths(depth, B, L, levels, msum):
    """Backward of the truncations over two letters where their wavefronts fill the chip, against the oracle."""
    ws, W = build_both("truncated", 2, depth=depth)
    ws.set_option("lanes", 1)
    ws.set_option("lanes_levels", levels)
    ws.set_option("chunks", 1)
    assert f"#define BACKWARD 1\n#define MSUM {msum}\n" in ws.jit_source(True, B)
    check_parity(ws, W, "truncated", depth, make_path("iid", 671, B, L, 2), make_grad_coeffs(672, B, ws.size),
                 sample=sorted({0, 1, B // 2, B - 2, B - 1}), what=f"two letters, depth {depth}, B={B}")


@pytest.mark.parametrize("d,depth,B,L,chunks", [
    (6, 5, 3, 21, 2),     # ragged last chunk
    (10, 4, 1, 50, 7),    # chunks of 8 segments, the last of 2
    (7, 3, 5, 64, 16),    # depth 3: products over single letters and pairs only; chunks of 4 segments
    (2, 7, 4, 100, 5),    # products of up to six cuts, slices of 64 words
    (9, 5, 1, 24, 3),     # 6,561 words of full length in a slice (512 threads), Q of 7,380 words
    (40, 3, 1, 32, 8),    # one word of length 1 and 40 of length 2 per slice
    (3, 8, 2, 33, 4),     # a chunk of 9 segments, the last of 6
    (12, 4, 2, 17, 2),    # the smallest length the launcher looks at is 16
    (6, 6, 2, 40, 0),     # the launcher's own choice (0), both directions
    (10, 4, 40, 70, 0),
    (5, 5, 9, 333, 0),
])
def test_time_chunks_of_truncations_with_lanes_as_words(d, depth, B, L, chunks, monkeypatch):
    """Time chunks of the word-per-lane truncations: chunk signatures, their products by first and last letter, the
    boundary adjoints and the walk over (path, chunk) rows, against the oracle; a call without a workspace walks whole
    paths and agrees to rounding (fp32 sums of L segments)."""
    import ctypes

    import torch
    monkeypatch.setenv("SIG_LANES", "1")
    ws, W = build_both("truncated", d, depth=depth)
    ws.set_option("chunks", chunks)
    X = make_path("iid", 171 + d, B, L, d)
    G = make_grad_coeffs(172 + d, B, ws.size)
    lib = S.load_library()
    if chunks:
        assert lib.sig_forward_workspace_bytes(ws._h, B, L + 1) >= 4 * B * 2 * ws.size  # room for two chunks at least
    check_parity(ws, W, "truncated", depth, X, G, what=f"time chunks, lanes = words, d={d} N={depth} C={chunks}")
    x = torch.from_numpy(X).cuda()
    c = S.sig_forward(ws, x)
    whole = torch.full_like(c, float("nan"))
    assert lib.sig_forward(ws._h, ctypes.c_void_p(x.data_ptr()), B, L + 1, ctypes.c_void_p(whole.data_ptr()), None, 0,
                           ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
    torch.cuda.synchronize()
    assert float((c - whole).norm() / whole.norm()) <= 1e-5


def nan_workspace(nbytes):
    """A float32 tensor of nbytes, 256-byte aligned, every entry NaN."""
    import torch
    buf = torch.full((nbytes // 4 + 64,), float("nan"), device="cuda")
    first = (-buf.data_ptr() % 256) // 4
    return buf[first:first + nbytes // 4]


@pytest.mark.parametrize("d,depth,B,L,chunks", [
    (6, 5, 3, 21, 2),
    (7, 3, 5, 64, 16),
    (2, 4, 9, 40, 5),     # a small truncation
    (12, 2, 3, 33, 4),    # depth 2: displacements
    (9, 5, 1, 24, 3),     # scan and adjoints of 512 threads
    (10, 5, 1, 17, 3),    # 10^4 words of full length in a slice: 1,024 threads
    (24, 4, 1, 16, 2),    # 24^3, the largest slice but one: 14 words a thread, 61 KB of LDS
])
def test_time_chunk_kernels_write_their_workspace(d, depth, B, L, chunks, monkeypatch):
    """The chunked calls of the word-per-lane truncations leave the chunk signatures (forward) and their products and
    boundary adjoints (backward) in the workspace; nothing of it is missing, and the results are the oracle's."""
    import torch
    monkeypatch.setenv("SIG_LANES", "1")
    ws, W = build_both("truncated", d, depth=depth)
    ws.set_option("chunks", chunks)
    X, G = make_path("iid", 471 + d, B, L, d), make_grad_coeffs(472 + d, B, ws.size)
    x, g = torch.from_numpy(X).cuda(), torch.from_numpy(G).cuda()
    lib = S.load_library()
    Lc = -(-L // chunks)
    C = -(-L // Lc)
    work = nan_workspace(int(lib.sig_forward_workspace_bytes(ws._h, B, L + 1)))
    c = S.sig_forward(ws, x, workspace=work)
    torch.cuda.synchronize()
    rows = work[:B * C * ws.size].reshape(B, C, ws.size)
    ws.set_option("chunks", 1)
    for k in range(C):
        part = S.sig_forward(ws, x[:, k * Lc:min((k + 1) * Lc, L) + 1].contiguous())
        assert float((rows[:, k] - part).norm() / part.norm()) <= 1e-5, k
    ws.set_option("chunks", chunks)
    low = int(ws.level_start[depth])
    work = nan_workspace(int(lib.sig_backward_workspace_bytes(ws._h, B, L + 1)))
    gp = S.sig_backward(ws, x, c, g, workspace=work)
    torch.cuda.synchronize()
    at = 0
    for n_rows in (C, C - 1, C - 1, C - 1):          # chunk signatures, products from the left, from the right, adjoints
        assert torch.isfinite(work[at:at + B * n_rows * low]).all(), (n_rows, at)
        at += -(-B * n_rows * low * 4 // 256) * 64
    errs = O.level_errors(c.cpu().numpy(), oracle_forward(X, W, "truncated", depth), np.array([len(w) for w in W]))
    assert max(errs.values()) <= FWD_TOL, errs
    assert O.grad_errors(gp.cpu().numpy(), oracle_backward(X, W, "truncated", depth, G.astype(np.float64))).max() <= BWD_TOL


def test_backward_with_the_workspace_of_whole_paths():
    """sig_backward takes time chunks where the workspace holds them; with the size a call over whole paths asks for it
    walks whole paths, leaves the workspace alone and agrees to rounding."""
    import torch
    d, depth, B, L = 9, 5, 1, 24
    ws, W = build_both("truncated", d, depth=depth)
    X, G = make_path("iid", 571, B, L, d), make_grad_coeffs(572, B, ws.size)
    x, g = torch.from_numpy(X).cuda(), torch.from_numpy(G).cuda()
    lib = S.load_library()
    c = S.sig_forward(ws, x)
    ws.set_option("chunks", 1)
    whole = int(lib.sig_backward_workspace_bytes(ws._h, B, L + 1))
    ws.set_option("chunks", 3)
    assert int(lib.sig_backward_workspace_bytes(ws._h, B, L + 1)) > whole
    work = nan_workspace(whole)
    gp = S.sig_backward(ws, x, c, g, workspace=work)
    torch.cuda.synchronize()
    assert torch.isnan(work).all()
    assert O.grad_errors(gp.cpu().numpy(), oracle_backward(X, W, "truncated", depth, G.astype(np.float64))).max() <= BWD_TOL
    with pytest.raises(S.SigError):
        S.sig_backward(ws, x, c, g, workspace=work[:whole // 4 - 64])


@pytest.mark.parametrize("d,depth,B,L,levels,split,backward_chunks", [
    (10, 4, 256, 35, 0, 2, None),      # halves of five children; 100 words in two wavefronts
    (7, 4, 500, 21, 0, 2, None),       # halves of four and three
    (9, 4, 3, 30, 2, 2, None),
    (6, 4, 1300, 5, 2, 1, None),       # as many wavefronts as SIMDs without halves
    (6, 5, 32, 60, 0, None, "R 2"),    # rows of two levels, signatures of 1,554 words in two wavefronts' LDS
    (10, 4, 2, 90, 0, None, "R 1"),    # one level, gradient sums as products
    (18, 3, 2, 64, 0, None, "R 1"),    # one level, sums by rows
    (2, 4, 5, 60, 0, None, "R 1"),     # 14 words, most of a row idle
    (4, 4, 5, 500, 0, None, None),     # many chunks
])
def test_forms_of_the_word_per_lane_kernels(d, depth, B, L, levels, split, backward_chunks):
    """Forward with the children of a word halved between two wavefronts, and the backward walk over the launcher's time chunks, whose
    lanes work out signature and adjoints at their chunk's end: against the oracle and, in other sums, against whole paths."""
    import torch
    ws, W = build_both("truncated", d, depth=depth)
    ws.set_option("lanes", 1)
    ws.set_option("lanes_levels", levels)
    if split:
        assert f"#define SP {split}\n" in ws.jit_source(False, B)
    lib = S.load_library()
    X = make_path("iid", 7600 + L, B, L, d)
    G = make_grad_coeffs(7700 + L, B, ws.size)
    x, g = torch.from_numpy(X).cuda(), torch.from_numpy(G).cuda()
    c = S.sig_forward(ws, x)
    low = int(ws.level_start[depth])
    work = nan_workspace(int(lib.sig_backward_workspace_bytes(ws._h, B, L + 1)))
    gp = S.sig_backward(ws, x, c, g, workspace=work)
    torch.cuda.synchronize()
    if backward_chunks:                                    # chunk signatures and nothing else in the workspace
        used = int(torch.isfinite(work).sum())
        C = used // (B * low)
        assert C > 1 and used == C * B * low and torch.isfinite(work[:used]).all()
        assert f"#define {backward_chunks}\n" in ws.jit_source(True, B * C)
    ws.set_option("chunks", 1)
    whole = S.sig_backward(ws, x, c, g)
    errs = O.level_errors(c.cpu().numpy(), oracle_forward(X, W, "truncated", depth), np.array([len(w) for w in W]))
    assert max(errs.values()) <= FWD_TOL, errs
    gref = oracle_backward(X, W, "truncated", depth, G.astype(np.float64))
    assert O.grad_errors(gp.cpu().numpy(), gref).max() <= BWD_TOL
    assert O.grad_errors(whole.cpu().numpy(), gref).max() <= BWD_TOL


@pytest.mark.parametrize("d,depth,B,L,levels,chunked", [
    (11, 3, 2, 1, 2, False),           # tiles of five segments: one, a whole tile, one more, several and a part
    (11, 3, 3, 5, 2, False),
    (12, 3, 2, 6, 2, False),
    (12, 3, 70, 13, 2, False),
    (11, 4, 2, 23, 2, False),          # 121 lanes in two wavefronts
    (12, 4, 1, 16, 2, False),          # 144 in three
    (11, 4, 64, 90, 0, True),          # the launcher's time chunks
    (12, 4, 64, 130, 0, True),
    (8, 4, 90, 130, 0, True),          # chunk signatures with a float between the runs: 8 lanes with one address in a bank each
    (4, 5, 200, 45, 0, True),          # .. of sixteen words
])
def test_backward_of_two_levels_in_partial_tiles_and_padded_chunk_signatures(d, depth, B, L, levels, chunked):
    """Two levels below a lane's word, backward: eleven and twelve letters, last tiles of every kind, and lanes that read chunk
    signatures in runs whose length is a multiple of sixteen; against the oracle."""
    import torch
    ws, W = build_both("truncated", d, depth=depth)
    ws.set_option("lanes", 1)
    ws.set_option("lanes_levels", levels)
    ws.set_option("chunks", 0 if chunked else 1)
    X = make_path("iid", 8100 + L, B, L, d)
    G = make_grad_coeffs(8200 + L, B, ws.size)
    x, g = torch.from_numpy(X).cuda(), torch.from_numpy(G).cuda()
    c = S.sig_forward(ws, x)
    low = int(ws.level_start[depth])
    work = nan_workspace(max(int(S.load_library().sig_backward_workspace_bytes(ws._h, B, L + 1)), 4))
    gp = S.sig_backward(ws, x, c, g, workspace=work)
    torch.cuda.synchronize()
    C = int(torch.isfinite(work).sum()) // (B * low)
    assert (C > 1) == chunked and "#define R 2\n" in ws.jit_source(True, B * max(C, 1))
    assert O.grad_errors(gp.cpu().numpy(), oracle_backward(X, W, "truncated", depth, G.astype(np.float64))).max() <= BWD_TOL


@pytest.mark.parametrize("d,depth,B,L,levels", [
    (11, 5, 2, 6, 2),           # 1,331 lanes, their first letters in runs over wavefronts, tiles of four segments
    (12, 5, 1, 9, 2),
    (11, 5, 16, 5, 0),          # the launcher's choice
    (11, 6, 1, 4, 2),           # tiles of three
])
def test_backward_of_two_levels_where_it_spills(d, depth, B, L, levels):
    """Two levels over eleven and twelve letters, deeper than the registers hold: the same against the oracle."""
    test_backward_of_two_levels_in_partial_tiles_and_padded_chunk_signatures(d, depth, B, L, levels, False)


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
@pytest.mark.parametrize("d,depth,L,levels,chunks", [
    (10, 4, 37, 1, 1),    # matrix-product sums, 16 wavefronts per path, ragged last tile
    (10, 4, 37, 1, 4),    # the same from the boundary adjoints of time chunks
    (3, 4, 20, 1, 1),     # 27 lanes: copies of the last word beyond them
    (16, 3, 9, 1, 1),     # every row of the product is a letter
    (6, 4, 18, 2, 1),     # two levels per lane: sums of rows
])
def test_non_finite_gradient_of_one_word_stays_with_its_letters(d, depth, L, levels, chunks, bad, monkeypatch):
    """d loss / dX of letter i sums over the words that contain i (Proposition 4.1).  An infinite or NaN upstream
    gradient of one word reaches the letters of that word in its path; the other letters and the other path have the
    gradient of the remaining words."""
    import torch
    monkeypatch.setenv("SIG_LANES", "1")
    monkeypatch.setenv("SIG_LANES_LEVELS", str(levels))
    ws, W = build_both("truncated", d, depth=depth)
    ws.set_option("chunks", chunks)
    X = make_path("iid", 371 + d, 2, L, d)
    G = make_grad_coeffs(372 + d, 2, ws.size)
    word = tuple(int(c) for c in np.random.default_rng(373).integers(0, 2, depth - 1)) + (2,)      # letters 0, 1 and 2 at most
    at = W.index(word)
    G[1, at] = 0.0
    ref = oracle_backward(X, W, "truncated", depth, G.astype(np.float64))
    G[1, at] = bad
    x = torch.from_numpy(X).cuda()
    g = S.sig_backward(ws, x, S.sig_forward(ws, x), torch.from_numpy(G).cuda()).cpu().numpy()
    others = [i for i in range(d) if i not in word]
    scale = np.abs(ref).max(axis=(1, 2))
    assert np.abs(g[0] - ref[0]).max() <= BWD_TOL * scale[0]
    assert not np.isfinite(g[1][:, sorted(set(word))]).any()
    if others:
        assert np.abs(g[1][:, others] - ref[1][:, others]).max() <= BWD_TOL * scale[1]


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
@pytest.mark.parametrize("d,depth,L,levels,length", [
    (10, 4, 90, 1, 3),    # one level, sums as products; a word of a lane's own
    (10, 4, 90, 1, 2),    # shared by ten lanes, of two wavefronts at times
    (10, 4, 90, 2, 4),    # two levels; a leaf
    (3, 4, 60, 1, 2),
    (16, 3, 64, 1, 3),
    (4, 6, 90, 0, 5),     # the fused kernel: eight chunks of a path in a workgroup
    (4, 6, 90, 0, 2),
    (4, 6, 40, 0, 6),
])
def test_non_finite_gradient_at_chunk_boundaries(d, depth, L, levels, length, bad, monkeypatch):
    """The same over the launcher's own time chunks, whose lanes work out the adjoints at the chunk ends: an infinite or NaN gradient
    of one word reaches its letters in its path and nothing else."""
    import torch
    if levels:
        monkeypatch.setenv("SIG_LANES", "1")
        monkeypatch.setenv("SIG_LANES_LEVELS", str(levels))
    ws, W = build_both("truncated", d, depth=depth)
    X, G = make_path("iid", 471 + L, 2, L, d), make_grad_coeffs(472 + L, 2, ws.size)
    word = tuple(int(c) for c in np.random.default_rng(473).integers(0, 2, length - 1)) + (2,)      # letters 0, 1 and 2 at most
    at = W.index(word)
    G[1, at] = 0.0
    ref = oracle_backward(X, W, "truncated", depth, G.astype(np.float64))
    G[1, at] = bad
    x, lib = torch.from_numpy(X).cuda(), S.load_library()
    work = nan_workspace(int(lib.sig_backward_workspace_bytes(ws._h, 2, L + 1)))
    g = S.sig_backward(ws, x, S.sig_forward(ws, x), torch.from_numpy(G).cuda(), workspace=work).cpu().numpy()
    if levels:                                                     # chunk signatures, and nothing else, in the workspace
        used, low = int(torch.isfinite(work).sum()), int(ws.level_start[depth])
        assert used > 2 * low and used % (2 * low) == 0
    else:
        assert ws.kernel_name(True, 2, L + 1) == "trunc_tails_bwd_kernel" and torch.isnan(work).all()
    others = [i for i in range(d) if i not in word]
    scale = np.abs(ref).max(axis=(1, 2))
    assert np.abs(g[0] - ref[0]).max() <= BWD_TOL * scale[0]
    assert not np.isfinite(g[1][:, sorted(set(word))]).any()
    assert np.abs(g[1][:, others] - ref[1][:, others]).max() <= BWD_TOL * scale[1]


@pytest.mark.parametrize("d,depth", [(3, 4), (4, 4), (10, 4)])
def test_chunk_boundaries_keep_the_precision_of_a_cancelling_gradient(d, depth):
    """The gradient of log-signature coordinates cancels in the adjoints of the short words.  Where the lanes work out the adjoints
    at a chunk's end, a word's shares are summed before the walk: within a wavefront (27 and 64 lanes a path) the error is that of
    the form with one value per word (geometric mean over 8 seeds; the sums differ in their order alone, 2 % measured, and without
    the sums it was 17 and 26 % larger), and with 1,000 lanes a path it stays below that of the walk over whole paths."""
    import torch
    lib = S.load_library()
    ws, W = build_both("truncated", d, depth=depth)
    wl = S.sig_wordset_build_logsig(d, depth)
    wl.upload("cuda:0")
    parent, letter, ls = wl.parent, wl.letter, wl.level_start
    words = []
    for i in range(wl.size):
        words.append((() if i < ls[2] else words[int(parent[i])]) + (int(letter[i]),))
    index = {w: i for i, w in enumerate(W)}
    at = torch.tensor([index[w] for w in words], device="cuda")
    low, B, L = int(ws.level_start[depth]), 4, 250
    errors = {"rule": [], "arrays": [], "whole": []}
    for seed in range(8):
        X = make_path("time0", 9100 + seed, B, L, d)
        x = torch.from_numpy(X).cuda()
        c = S.sig_forward(ws, x)
        n_lyn = int(lib.sig_wordset_n_lyndon(wl._h))
        gl = torch.from_numpy(make_grad_coeffs(9200 + seed, B, n_lyn)).cuda()
        g = torch.zeros_like(c)
        g[:, at] = S.sig_logsig_backward(wl, c[:, at].contiguous(), gl)
        ref = oracle_backward(X, W, "truncated", depth, g.cpu().numpy().astype(np.float64))
        ws.set_option("chunks", 0)
        work = nan_workspace(int(lib.sig_backward_workspace_bytes(ws._h, B, L + 1)))
        out = {"rule": S.sig_backward(ws, x, c, g, workspace=work)}
        torch.cuda.synchronize()
        C = int(torch.isfinite(work).sum()) // (B * low)
        assert C > 1
        for name, chunks in (("arrays", C), ("whole", 1)):
            ws.set_option("chunks", chunks)
            out[name] = S.sig_backward(ws, x, c, g)
        for name, gp in out.items():
            errors[name].append(np.linalg.norm(gp.cpu().numpy() - ref) / np.linalg.norm(ref))
    mean = {name: float(np.exp(np.mean(np.log(e)))) for name, e in errors.items()}
    assert mean["rule"] <= mean["whole"], mean
    if d ** (depth - 1) <= 64:
        assert mean["rule"] <= 1.1 * mean["arrays"], mean


@pytest.mark.parametrize("d,depth,B,L,lanes_are_words", [
    (2, 4, 32, 64, True),       # 8 lanes per path; chunks
    (2, 4, 64, 64, False),      # paths that fill a wavefront, and short
    (2, 4, 64, 65, True),
    (3, 4, 5, 15, True),        # too short for chunks
    (2, 5, 769, 70, False),     # many paths
    (3, 3, 70, 33, True),
    (5, 3, 1025, 17, False),
    (2, 2, 3, 40, True),        # depth 2: the chunk signatures over single letters are displacements
    (12, 2, 9, 50, True),
    (31, 2, 2, 21, True),       # the largest alphabet whose letters leave half a wavefront empty
    (12, 2, 4, 1, True),        # a single segment
])
def test_small_truncations_with_few_paths(d, depth, B, L, lanes_are_words):
    """Truncations whose words fill less than half a wavefront: a word per lane with time chunks while the paths are
    few, a path per lane beyond; both sides of the line against the oracle.  A forward call without a workspace is
    refused on either side, and the entry point without a workspace runs after one sig_backward call."""
    import ctypes

    import torch
    ws, W = build_both("truncated", d, depth=depth)
    assert ws.kernel_name(False, B, L + 1) == ("sig_fwd_lanes" if lanes_are_words else "sig_fwd_jit")
    X = make_path("iid", 271 + d, B, L, d)
    G = make_grad_coeffs(272 + d, B, ws.size)
    check_parity(ws, W, "truncated", depth, X, G, what=f"small truncation d={d} N={depth} B={B} L={L}")
    x, g = torch.from_numpy(X).cuda(), torch.from_numpy(G).cuda()
    c = torch.empty((B, ws.size), device="cuda")
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    assert S.load_library().sig_forward(ws._h, ctypes.c_void_p(x.data_ptr()), B, L + 1, ctypes.c_void_p(c.data_ptr()), None, 0,
                                        stream) == -5
    c = S.sig_forward(ws, x)
    a, b = S.sig_backward(ws, x, c, g), S.sig_backward_static(ws, x, c, g, torch.empty_like(x))
    torch.cuda.synchronize()
    assert O.grad_errors(b.cpu().numpy(), a.cpu().numpy().astype(np.float64)).max() <= BWD_TOL


def test_lanes_as_words_on_a_long_path():
    """5,000 segments through the word-per-lane kernels: many staging tiles, and the reconstruction of the
    backward pass over a long walk (within the gradient tolerance, as for the 4,096 segments of c5)."""
    ws, W = build_both("truncated", 6, depth=4)
    B, L = 2, 5000
    assert ws.kernel_name(True, B, L + 1) == "sig_bwd_lanes"
    X = make_path("iid", 91, B, L, 6)
    G = make_grad_coeffs(92, B, ws.size)
    check_parity(ws, W, "truncated", 4, X, G, what="lanes = words, 5,000 segments")


def test_lanes_as_words_on_random_shapes(monkeypatch):
    """Sixteen seeded random shapes (2..20 letters, depth 2..6, up to 30,000 words, 1..5 paths of 1..40 segments),
    alternating between the two forms of the word-per-lane kernels where both exist."""
    rng = np.random.default_rng(2024)
    monkeypatch.setenv("SIG_LANES", "1")
    done = 0
    while done < 16:
        d, depth = int(rng.integers(2, 21)), int(rng.integers(2, 7))
        if sum(d ** n for n in range(1, depth + 1)) > 30000 or (d, depth) in ((4, 6), (8, 5), (16, 4)):
            continue
        B, L = int(rng.integers(1, 6)), int(rng.integers(1, 41))
        monkeypatch.setenv("SIG_LANES_LEVELS", str(1 + done % 2))
        ws, W = build_both("truncated", d, depth=depth)
        assert ws.kernel_name(True, B, L + 1) == "sig_bwd_lanes"
        X = make_path("iid", 300 + done, B, L, d)
        G = make_grad_coeffs(400 + done, B, ws.size)
        check_parity(ws, W, "truncated", depth, X, G, what=f"random shape {done}: d={d} N={depth} B={B} L={L}")
        done += 1


def test_lanes_as_words_and_lanes_as_paths_agree(monkeypatch):
    """The two run-time compiled forms of one truncation on the same inputs (each is compared with the oracle
    elsewhere; this pins the switch between them)."""
    import torch
    d, depth, B, L = 6, 4, 70, 40
    X = torch.from_numpy(make_path("iid", 81, B, L, d)).cuda()
    out = {}
    for form in ("0", "1"):
        monkeypatch.setenv("SIG_LANES", form)
        ws = S.sig_wordset_build_truncated(d, depth)
        ws.upload("cuda:0")
        assert ws.kernel_name(False, B, L + 1) == ("sig_fwd_lanes" if form == "1" else "sig_fwd_jit")
        G = torch.from_numpy(make_grad_coeffs(82, B, ws.size)).cuda()
        c = S.sig_forward(ws, X)
        g = S.sig_backward(ws, X, c, G)
        out[form] = (c.cpu().numpy(), g.cpu().numpy())
    np.testing.assert_allclose(out["0"][0], out["1"][0], rtol=2e-4, atol=1e-6)
    np.testing.assert_allclose(out["0"][1], out["1"][1], rtol=1e-3, atol=1e-4)


def test_graph_induced_word_set():
    edges = [(0, 1), (0, 2), (1, 3), (2, 3), (3, 4), (3, 5), (1, 5), (4, 5), (2, 4)]
    ws = S.sig_wordset_build_graph(6, edges, 5)
    ws.upload("cuda:0")
    W = O.graph_words(6, edges, 5)
    assert ws.size == len(W)
    X = make_path("iid", 61, 70, 33, 6)
    G = make_grad_coeffs(62, 70, ws.size)
    check_parity(ws, W, "words", None, X, G, what="graph-induced set")


def test_leadlag_transform_and_sparse_word_set():
    import torch
    d, depth, B, n = 3, 4, 9, 12
    X = make_path("iid", 63, B, n - 1, d)
    xp = torch.from_numpy(X).cuda()
    yp = S.sig_leadlag_transform(xp)
    Y = O.leadlag_transform(X)
    assert np.array_equal(yp.cpu().numpy(), Y)                       # copies only: exact
    # its adjoint against the transpose of the (linear) oracle transform, applied to a random cotangent
    Gy = np.random.default_rng(64).standard_normal(Y.shape).astype(np.float32)
    gx = S.sig_leadlag_backward(torch.from_numpy(Gy).cuda()).cpu().numpy()
    ref = np.zeros(X.shape, dtype=np.float64)
    ref += Gy[:, 0::2, :d] + Gy[:, 0::2, d:]
    ref[:, :-1] += Gy[:, 1::2, :d]
    ref[:, 1:] += Gy[:, 1::2, d:]
    np.testing.assert_allclose(gx, ref, rtol=1e-6, atol=1e-6)
    # signatures of the lead-lag path on the sparse set
    ws = S.sig_wordset_build_leadlag_sparse(d, depth)
    ws.upload("cuda:0")
    W = O.prefix_closure(O.leadlag_sparse_words(d, depth))
    assert ws.size == len(W)
    G = make_grad_coeffs(65, B, ws.size)
    check_parity(ws, W, "words", None, Y, G, what="sparse lead-lag set")


WINDOW_SETS = [
    ("truncated", dict(d=3, depth=4)),
    ("truncated", dict(d=4, depth=6)),
    ("truncated", dict(d=5, depth=4)),
    ("truncated", dict(d=6, depth=4)),           # a word per lane: 36 words of length 2
    ("truncated", dict(d=3, depth=6)),           # a word per lane: 81 words of length 4, two wavefronts per row
    ("anisotropic", dict(d=4, weights=(1.0, 1.0, 2.0, 3.0), cutoff=5.0)),
    ("words", dict(d=6, n_words=500, max_len=5)),
]


# table_driven: the fallback kernels, whose windows are gathered into padded sub-paths and scattered back
@pytest.mark.parametrize("case,B,table_driven",
                         [(c, B, False) for c in range(len(WINDOW_SETS)) for B in (5, 13)] +
                         [(c, 5, True) for c, (kind, kw) in enumerate(WINDOW_SETS) if (kw["d"], kw.get("depth")) != (4, 6)])
def test_windows(case, B, table_driven):
    """Signatures over user-given windows (expanding, sliding, overlapping, single-segment, empty, whole path) against
    one oracle evaluation per window, forward and backward."""
    import torch
    kind, kw = WINDOW_SETS[case]
    d = kw["d"]
    words = random_prefix_closed_words(400 + case, d, kw["n_words"], kw["max_len"]) if kind == "words" else None
    ws, W = build_both(kind, d, depth=kw.get("depth"), weights=kw.get("weights"), cutoff=kw.get("cutoff"), words=words)
    if table_driven:
        ws.set_option("no_jit", 1)                 # (d = 4, depth 6 has a precompiled kernel and is left out above)
        assert ws.kernel_name(True, B * 11, 41) == "bwd_generic_kernel"
    if not table_driven and kind == "truncated" and (d, kw["depth"]) in ((6, 4), (3, 6)):
        assert ws.kernel_name(True, B * 11, 41) == "sig_bwd_lanes"
    L = 40                      # B = 13: 143 (path, window) rows, more than two wavefronts of rows for the lane = row kernels
    X = make_path("iid", 410 + case, B, L, d)
    windows = [(0, L), (0, 1), (0, 7), (0, 23), (5, 15), (10, 20), (15, 25), (39, 40), (17, 17), (3, 38), (5, 15)]
    K = len(windows)
    G = make_grad_coeffs(420 + case, B * K, ws.size).reshape(B, K, ws.size)
    xp = torch.from_numpy(X).cuda()
    coeffs = S.sig_forward_windows(ws, xp, windows)
    gp = S.sig_backward_windows(ws, xp, windows, coeffs, torch.from_numpy(G).cuda())
    torch.cuda.synchronize()
    coeffs, gp = coeffs.cpu().numpy(), gp.cpu().numpy()
    ref = O.forward_windows(X, W, windows)
    lengths = np.array([len(w) for w in W])
    for k, (l, r) in enumerate(windows):
        if l == r:
            assert np.all(coeffs[:, k] == 0.0)
            continue
        for n, e in O.level_errors(coeffs[:, k], ref[:, k], lengths).items():
            assert e <= FWD_TOL, f"window {k} level {n}: {e:.3e}"
    gref = O.backward_windows(X, W, windows, G.astype(np.float64))
    assert O.grad_errors(gp, gref).max() <= BWD_TOL


@pytest.mark.parametrize("d,depth,B,L", [(2, 6, 7, 20), (3, 4, 66, 15), (4, 5, 3, 9), (5, 1, 2, 4), (4, 6, 5, 33)])
def test_log_signature(d, depth, B, L):
    """Log-signature in Lyndon-word coordinates: signature on the reduced word set, then the tensor logarithm word by
    word, against the oracle's dense tensor logarithm of the full truncated signature."""
    import torch
    ws = S.sig_wordset_build_logsig(d, depth)
    ws.upload("cuda:0")
    X = make_path("iid", 500 + d, B, L, d)
    xp = torch.from_numpy(X).cuda()
    coeffs = S.sig_forward(ws, xp)
    lg = S.sig_logsig_forward(ws, coeffs).cpu().numpy()
    ref = O.logsig_from_path(X, depth)
    lyn = O.lyndon_words(d, depth)
    assert lg.shape == ref.shape == (B, len(lyn))
    lengths = np.array([len(w) for w in lyn])
    for n, e in O.level_errors(lg, ref, lengths).items():
        assert e <= FWD_TOL, f"log-signature level {n}: {e:.3e}"


@pytest.mark.parametrize("d,depth,B", [(4, 6, 68), (4, 6, 256), (4, 6, 257), (8, 4, 65), (26, 3, 12), (3, 6, 256)])
def test_log_signature_of_a_path_in_lds(d, depth, B):
    """Forward with a workgroup's path in LDS (65,536 words and more, up to 256 paths; more Lyndon words than threads among them) and the
    forms beside it: a path's coordinates are the same whichever form the batch takes."""
    import torch
    ws = S.sig_wordset_build_logsig(d, depth).upload("cuda:0")
    gen = torch.Generator(device="cuda").manual_seed(900 + B)
    c = torch.randn((B, ws.size), generator=gen, device="cuda")
    out = S.sig_logsig_forward(ws, c)
    for b in (0, B // 2, B - 1):
        one = S.sig_logsig_forward(ws, c[b:b + 1])             # places by word, read from memory
        assert torch.allclose(out[b], one[0], rtol=1e-5, atol=1e-5 * float(one.abs().max()))


@pytest.mark.parametrize("d,depth,B", [
    (25, 3, 12), (5, 5, 80), (5, 5, 79),        # depth below the kernel's bound; 79 paths have 65,491 words
    (40, 3, 3),                                 # 92 KB a path
])
def test_log_signature_up_to_the_limits_of_a_path_in_lds(d, depth, B):
    """Words shorter than the kernel is made for, and the row and word counts its rule ends at."""
    test_log_signature_of_a_path_in_lds(d, depth, B)


@pytest.mark.parametrize("d,depth,B,L", [(5, 5, 80, 6), (26, 3, 12, 5), (25, 3, 12, 5), (8, 4, 65, 7)])
def test_log_signature_of_many_words(d, depth, B, L):
    """65,536 words and more in a batch, which a workgroup's path in LDS serves (26 letters: too long a row), against the oracle."""
    test_log_signature(d, depth, B, L)


@pytest.mark.parametrize("d,depth,B", [
    (4, 6, 3),       # 964 Lyndon words of up to six letters: contributions and coefficients of a path in 103 KB of LDS
    (5, 1, 2),       # letters only: no list of the inverse table is long
    (3, 3, 65),
    (2, 7, 2),       # pairs beyond a word's length
    (2, 9, 1),       # words of more than eight letters (tables in scratch memory)
    (6, 4, 5),       # the reduced word set: words of full length are Lyndon words
    (5, 5, 2),
    (6, 5, 1),       # contributions too large for LDS: the gradient row alone is kept there
])
def test_log_signature_adjoint_forms_agree(d, depth, B):
    """The adjoint of the tensor logarithm in the form that keeps a path's contributions in LDS (or the one that adds into
    the gradient row there) against the form that writes them out and gathers them: the same terms in another order, so
    sums of at most a few thousand fp32 terms."""
    import torch
    ws = S.sig_wordset_build_logsig(d, depth)
    ws.upload("cuda:0")
    n_lyn = int(S.load_library().sig_wordset_n_lyndon(ws._h))
    gen = torch.Generator(device="cuda").manual_seed(600 + 10 * d + depth)
    c = torch.randn((B, ws.size), generator=gen, device="cuda")
    g = torch.randn((B, n_lyn), generator=gen, device="cuda")
    one = S.sig_logsig_backward(ws, c, g)
    ws.set_option("logsig_gather", 1)
    two = S.sig_logsig_backward(ws, c, g)
    torch.cuda.synchronize()
    assert torch.isfinite(one).all()
    assert float((one.double() - two.double()).norm() / two.double().norm()) <= 2e-6


@pytest.mark.parametrize("d,depth,B,n_lyndon", [
    (4, 4, 3, 90),                          # few words: atomics
    (5, 4, 512, 205), (5, 4, 513, 205),     # around 200: by the number of paths
    (9, 3, 2, 285), (2, 10, 600, 226),
    (20, 2, 4, 210), (31, 2, 512, 496), (31, 2, 513, 496), (36, 2, 2, 666),      # pairs of letters
])
def test_log_signature_adjoint_on_either_side_of_its_lines(d, depth, B, n_lyndon):
    """The forms of the log-signature adjoint by the number of Lyndon words, against the form that gathers (the same terms in
    another order)."""
    import torch
    ws = S.sig_wordset_build_logsig(d, depth).upload("cuda:0")
    assert int(S.load_library().sig_wordset_n_lyndon(ws._h)) == n_lyndon
    gen = torch.Generator(device="cuda").manual_seed(700 + 10 * d + depth)
    c, g = torch.randn((B, ws.size), generator=gen, device="cuda"), torch.randn((B, n_lyndon), generator=gen, device="cuda")
    one = S.sig_logsig_backward(ws, c, g)
    ws.set_option("logsig_gather", 1)
    two = S.sig_logsig_backward(ws, c, g)
    torch.cuda.synchronize()
    assert float((one.double() - two.double()).norm() / two.double().norm()) <= 2e-6


@pytest.mark.parametrize("d,depth", [(4, 4), (3, 6), (2, 8), (2, 9), (5, 1)])
def test_log_signature_tables_by_word_and_by_pair(d, depth):
    """Few and many Lyndon words of a call read their places in another order (from 65,536 on): the same arithmetic."""
    import torch
    ws = S.sig_wordset_build_logsig(d, depth).upload("cuda:0")
    n_lyn = int(S.load_library().sig_wordset_n_lyndon(ws._h))
    B = -(-65536 // n_lyn)
    c = torch.randn((B, ws.size), generator=torch.Generator(device="cuda").manual_seed(800 + d), device="cuda")
    many = S.sig_logsig_forward(ws, c)
    few = torch.cat([S.sig_logsig_forward(ws, c[:B // 2]), S.sig_logsig_forward(ws, c[B // 2:])])
    assert torch.equal(many, few)


@pytest.mark.parametrize("d,B,L", [
    (2, 65, 31), (2, 1, 33),        # tiles of 32 segments: one short, one with a second tile of one segment
    (7, 130, 9), (7, 64, 10),       # 63 of 64 floats of a tile row in use
    (33, 3, 2),                     # a segment per tile
    (48, 66, 3),                    # the largest alphabet of the specialised backward kernels
])
def test_transposed_increments_and_gradients(d, B, L):
    """The transposition around the specialised kernels at the edges of its tiles (floor(64 / d) segments x 64 rows),
    whole paths and, on the same set, windows of unequal length (rows that end inside a tile or have no segment)."""
    import torch
    words = random_prefix_closed_words(700 + d, d, 40, 6 if d == 2 else 3)
    ws, W = build_both("words", d, words=words)
    assert ws.kernel_name(False, B, L + 1) == "sig_fwd_jit"
    X = make_path("iid", 701 + d, B, L, d)
    G = make_grad_coeffs(702 + d, B, ws.size)
    check_parity(ws, W, "words", None, X, G, what=f"d={d} B={B} L={L}")
    wins = [(0, L), (L // 2, L), (0, 1), (L, L)]
    x = torch.from_numpy(X).cuda()
    c = S.sig_forward_windows(ws, x, wins)
    g = torch.from_numpy(make_grad_coeffs(703 + d, B * len(wins), ws.size).reshape(B, len(wins), ws.size)).cuda()
    gp = S.sig_backward_windows(ws, x, wins, c, g)
    total = torch.zeros_like(x)
    for k, (l, r) in enumerate(wins):
        sub = x[:, l:r + 1].contiguous()
        ck = S.sig_forward(ws, sub)
        assert torch.allclose(ck, c[:, k], rtol=1e-5, atol=1e-6)
        total[:, l:r + 1] += S.sig_backward(ws, sub, ck, g[:, k].contiguous())
    torch.cuda.synchronize()
    assert O.grad_errors(gp.cpu().numpy(), total.cpu().numpy().astype(np.float64)).max() <= BWD_TOL


@pytest.mark.parametrize("d,n_words,B,L,rounds", [
    (7, 300, 70, 13, 1),       # 42 rows a tile: ten whole rounds of four wavefronts and two rows
    (14, 300, 65, 7, 1),       # tiles of three segments, the last ragged
    (48, 300, 3, 2, 1),        # one segment a tile
    (7, 1000, 2497, 7, 0),     # two workgroups per compute unit, the last group one path
    (5, 1000, 2497, 9, 2),     # tiles of eight segments
    (3, 4, 5, 9, 1),           # units of one word
])
def test_gradient_tile_sums(d, n_words, B, L, rounds):
    """The specialised backward with the sum of its gradient tiles as a function and inlined, against the oracle."""
    words = random_prefix_closed_words(720, d, n_words, 5)
    ws, W = build_both("words", d, words=words)
    assert f"#define FLUSH_ROUNDS {rounds}\n" in ws.jit_source(True, B)
    check_parity(ws, W, "words", None, make_path("iid", 721, B, L, d), make_grad_coeffs(722, B, ws.size),
                 sample=None if B < 100 else list(range(0, B, 208)), what=f"B={B} L={L}")


@pytest.mark.parametrize("two_kernels", [False, True])
def test_log_signature_gradient(monkeypatch, two_kernels):
    """d <G, logsig(X)> / dX through sig_logsig_backward and sig_backward against central differences of the oracle;
    sig_logsig_backward in its one-kernel form (gradient row summed in LDS) and in the form for rows that do not fit
    there (contributions written out, then gathered per word)."""
    import torch
    if two_kernels:
        monkeypatch.setenv("SIG_LOGSIG_GATHER", "1")
    else:
        monkeypatch.delenv("SIG_LOGSIG_GATHER", raising=False)
    d, depth, B, L = 3, 4, 2, 5
    ws = S.sig_wordset_build_logsig(d, depth)
    ws.upload("cuda:0")
    # points on a grid of 2^-6, so that X +- h is exact in fp32 (the oracle consumes fp32 paths)
    X = (np.round(make_path("iid", 510, B, L, d) * 64.0) / 64.0).astype(np.float32)
    G = np.random.default_rng(511).standard_normal((B, int(S.load_library().sig_wordset_n_lyndon(ws._h)))).astype(np.float32)
    xp = torch.from_numpy(X).cuda()
    coeffs = S.sig_forward(ws, xp)
    gc = S.sig_logsig_backward(ws, coeffs, torch.from_numpy(G).cuda())
    gp = S.sig_backward(ws, xp, coeffs, gc).cpu().numpy()
    Xd = X.astype(np.float64)
    fun = lambda Y: float((O.logsig_from_path(Y, depth) * G).sum())
    num = np.zeros_like(Xd)
    h = 2.0 ** -10
    for idx in np.ndindex(*Xd.shape):
        Yp, Ym = Xd.copy(), Xd.copy()
        Yp[idx] += h
        Ym[idx] -= h
        num[idx] = (fun(Yp) - fun(Ym)) / (2 * h)
    assert O.grad_errors(gp, num).max() <= BWD_TOL


@pytest.mark.parametrize("kind,d,depth,B,L", [("truncated", 4, 6, 9, 70), ("truncated", 8, 5, 2, 24), ("words", 5, 4, 70, 19),
                                              ("truncated", 6, 4, 5, 31)])
def test_step_captured_in_a_graph(kind, d, depth, B, L):
    """Forward + backward recorded into a HIP graph (the library enqueues kernels only: no allocation, no memset) and
    replayed on new inputs, with eager calls and synchronisations between the replays; every replay must reproduce
    the eager results, and the first one the oracle's."""
    import torch
    from sig_workloads import random_prefix_closed_words
    words = random_prefix_closed_words(1699, d, 200, depth) if kind == "words" else None
    ws, W = build_both(kind, d, depth=depth, words=words)
    lib = S.load_library()
    X0 = make_path("iid", 1700, B, L, d)
    G0 = make_grad_coeffs(1701, B, ws.size)
    xp = torch.from_numpy(X0).cuda()
    grad = torch.from_numpy(G0).cuda()
    coeffs = torch.empty((B, ws.size), dtype=torch.float32, device="cuda")
    gpath = torch.empty((B, L + 1, d), dtype=torch.float32, device="cuda")
    wf = torch.empty(max(int(lib.sig_forward_workspace_bytes(ws._h, B, L + 1)), 256), dtype=torch.uint8, device="cuda")
    wb = torch.empty(max(int(lib.sig_backward_workspace_bytes(ws._h, B, L + 1)), 256), dtype=torch.uint8, device="cuda")

    def step():
        S.sig_forward(ws, xp, out=coeffs, workspace=wf)
        S.sig_backward(ws, xp, coeffs, grad, out=gpath, workspace=wb)

    step()                                   # compiles / sets kernel attributes outside the capture
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    lengths = np.array([len(w) for w in W])
    for rep in range(3):
        X = make_path("iid", 1710 + rep, B, L, d)
        G = make_grad_coeffs(1720 + rep, B, ws.size)
        xp.copy_(torch.from_numpy(X).cuda())
        grad.copy_(torch.from_numpy(G).cuda())
        coeffs.zero_()
        gpath.zero_()
        graph.replay()
        torch.cuda.synchronize()
        c_graph, g_graph = coeffs.cpu().numpy(), gpath.cpu().numpy()
        c_eager = S.sig_forward(ws, xp)
        g_eager = S.sig_backward(ws, xp, c_eager, grad)
        torch.cuda.synchronize()
        assert np.array_equal(c_graph, c_eager.cpu().numpy()), f"replay {rep}: forward differs from the eager call"
        assert O.grad_errors(g_graph, g_eager.cpu().numpy().astype(np.float64)).max() <= 1e-5, f"replay {rep}"
        if rep == 0:
            for n, e in O.level_errors(c_graph, O.forward_words(X, W), lengths).items():
                assert e <= FWD_TOL, (n, e)
            assert O.grad_errors(g_graph, O.backward_words(X, W, G.astype(np.float64))).max() <= BWD_TOL


@pytest.mark.parametrize("kind,d,depth,B,L", [("anisotropic", 3, None, 5, 200), ("anisotropic", 3, None, 3, 130), ("truncated", 8, 5, 2, 200)])
def test_checkpointed_step_captured_in_a_graph(kind, d, depth, B, L):
    """The pair of calls that keeps the time-chunk signatures, recorded into a HIP graph with its checkpoint and
    workspaces (kernels only: the clearing is a kernel, the products and boundary adjoints are kernels) and replayed
    on new inputs with eager work between the replays."""
    import torch
    ws, W = build_both(kind, d, depth=depth, weights=(1.0, 1.25, 1.5), cutoff=4.5)
    if kind == "anisotropic":
        ws.set_option("ckpt_chunks", 3 if L >= 192 else 2)
    lib = S.load_library()
    nck = int(lib.sig_checkpoint_bytes(ws._h, B, L + 1))
    assert nck > 0
    xp = torch.from_numpy(make_path("iid", 1800, B, L, d)).cuda()
    grad = torch.from_numpy(make_grad_coeffs(1801, B, ws.size)).cuda()
    coeffs = torch.empty((B, ws.size), dtype=torch.float32, device="cuda")
    gpath = torch.empty((B, L + 1, d), dtype=torch.float32, device="cuda")
    ck = torch.empty(nck, dtype=torch.uint8, device="cuda")
    wf = torch.empty(max(int(lib.sig_forward_checkpointed_workspace_bytes(ws._h, B, L + 1)), 256), dtype=torch.uint8, device="cuda")
    wb = torch.empty(max(int(lib.sig_backward_checkpointed_workspace_bytes(ws._h, B, L + 1)), 256), dtype=torch.uint8, device="cuda")

    def step():
        S.sig_forward_checkpointed(ws, xp, out=coeffs, checkpoint=ck, workspace=wf)
        S.sig_backward_checkpointed(ws, xp, coeffs, grad, ck, out=gpath, workspace=wb)

    step()                                   # compiles / sets kernel attributes outside the capture
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    lengths = np.array([len(w) for w in W])
    for rep in range(3):
        X = make_path("iid", 1810 + rep, B, L, d)
        G = make_grad_coeffs(1820 + rep, B, ws.size)
        xp.copy_(torch.from_numpy(X).cuda())
        grad.copy_(torch.from_numpy(G).cuda())
        coeffs.zero_()
        gpath.fill_(7.0)
        ck.zero_()
        graph.replay()
        torch.cuda.synchronize()
        c_graph, g_graph = coeffs.cpu().numpy(), gpath.cpu().numpy()
        c_eager, ck_eager = S.sig_forward_checkpointed(ws, xp)
        g_eager = S.sig_backward_checkpointed(ws, xp, c_eager, grad, ck_eager)
        torch.cuda.synchronize()
        assert np.array_equal(c_graph, c_eager.cpu().numpy()), f"replay {rep}: forward differs from the eager call"
        assert O.grad_errors(g_graph, g_eager.cpu().numpy().astype(np.float64)).max() <= 1e-5, f"replay {rep}"
        if rep == 0:
            ref = O.forward_dense(X, depth) if kind == "truncated" else O.forward_words(X, W)
            for n, e in O.level_errors(c_graph, ref, lengths).items():
                assert e <= FWD_TOL, (n, e)
            gref = O.backward_dense(X, depth, G.astype(np.float64)) if kind == "truncated" else O.backward_words(X, W, G.astype(np.float64))
            assert O.grad_errors(g_graph, gref).max() <= BWD_TOL


@pytest.mark.parametrize("chunks,kept", [(0, False), (1, True)])
def test_checkpointed_backward_of_few_paths_of_a_word_set(chunks, kept):
    """On few paths the backward call takes more chunks than the checkpoint holds and works out their signatures itself: seen by a
    checkpoint of NaN that it does not read.  With the option "chunks" = 1 there are no others, and the kept ones are used."""
    import torch
    B, L = 3, 400
    ws, W = build_both("anisotropic", 3, weights=(1.0, 1.25, 1.5), cutoff=4.5)
    ws.set_option("chunks", chunks)
    X, G = make_path("iid", 1900, B, L, 3), make_grad_coeffs(1901, B, ws.size)
    x, g = torch.from_numpy(X).cuda(), torch.from_numpy(G).cuda()
    c, ck = S.sig_forward_checkpointed(ws, x)
    assert ck.numel() > 0
    gref = O.backward_words(X, W, G.astype(np.float64))
    gp = S.sig_backward_checkpointed(ws, x, c, g, ck)
    assert O.grad_errors(gp.cpu().numpy(), gref).max() <= BWD_TOL
    ck.view(torch.float32).fill_(float("nan"))
    gp = S.sig_backward_checkpointed(ws, x, c, g, ck).cpu().numpy()
    assert np.isnan(gp).any() if kept else O.grad_errors(gp, gref).max() <= BWD_TOL


def test_checkpointed_backward_captured_after_an_eager_forward():
    """The forward call of a checkpointed pair loads the kernels of the backward call, also of one that takes other chunks than are
    kept: recorded alone, after nothing but an eager forward call, it replays to the oracle's gradient."""
    import torch
    B, L = 3, 400
    ws, W = build_both("anisotropic", 3, weights=(1.0, 1.25, 1.5), cutoff=4.5)
    x = torch.from_numpy(make_path("iid", 1910, B, L, 3)).cuda()
    g = torch.from_numpy(make_grad_coeffs(1911, B, ws.size)).cuda()
    c, ck = S.sig_forward_checkpointed(ws, x)
    lib = S.load_library()
    wb = torch.empty(int(lib.sig_backward_checkpointed_workspace_bytes(ws._h, B, L + 1)), dtype=torch.uint8, device="cuda")
    gp = torch.empty_like(x)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        S.sig_backward_checkpointed(ws, x, c, g, ck, out=gp, workspace=wb)
    for rep in range(3):
        X, G = make_path("iid", 1920 + rep, B, L, 3), make_grad_coeffs(1930 + rep, B, ws.size)
        x.copy_(torch.from_numpy(X))
        g.copy_(torch.from_numpy(G))
        S.sig_forward_checkpointed(ws, x, out=c, checkpoint=ck)
        gp.fill_(7.0)
        graph.replay()
        torch.cuda.synchronize()
        assert O.grad_errors(gp.cpu().numpy(), O.backward_words(X, W, G.astype(np.float64))).max() <= BWD_TOL, rep


def test_suffix_closed_sets_accept_the_workspace_of_their_own_chunks():
    """Small launches of a set closed under suffixes are told the workspace of their finer chunks.  What the chunks of the
    checkpointed calls need is accepted as well, by all four calls, and a byte less refused."""
    import ctypes
    import torch
    d, B, L, C = 3, 512, 512, 4
    ws, W = build_both("anisotropic", d, weights=(1.0, 1.25, 1.5), cutoff=4.5)
    ws.set_option("ckpt_chunks", C)
    lib = S.load_library()
    X, G = make_path("iid", 5400, B, L, d), make_grad_coeffs(5401, B, ws.size)
    x, g = torch.from_numpy(X).cuda(), torch.from_numpy(G).cuda()
    c, gp = torch.empty((B, ws.size), device="cuda"), torch.empty_like(x)
    rows = B * C // 64 * (L // C) * d * 64 * 4                     # transposed increments of the chunks
    arrays = int(lib.sig_checkpoint_bytes(ws._h, B, L + 1))
    assert arrays == (4 * B * C * ws.size + 255) // 256 * 256
    ck = torch.empty(arrays, dtype=torch.uint8, device="cuda")
    work = torch.empty(2 * rows + 3 * arrays, dtype=torch.uint8, device="cuda")
    P = ctypes.c_void_p
    xp, cp, gr, out, kp, wk = (P(t.data_ptr()) for t in (x, c, g, gp, ck, work))
    st = P(torch.cuda.current_stream().cuda_stream)
    few = slice(0, 3)
    ref = O.forward_words(X[few], W)
    gref = O.backward_words(X[few], W, G[few].astype(np.float64))
    lengths = np.array([len(w) for w in W])
    calls = [
        (rows + arrays, lib.sig_forward_workspace_bytes, lambda n: lib.sig_forward(ws._h, xp, B, L + 1, cp, wk, n, st)),
        (2 * rows + 3 * arrays, lib.sig_backward_workspace_bytes,
         lambda n: lib.sig_backward(ws._h, xp, cp, gr, B, L + 1, out, wk, n, st)),
        (rows, lib.sig_forward_checkpointed_workspace_bytes,
         lambda n: lib.sig_forward_checkpointed(ws._h, xp, B, L + 1, cp, kp, arrays, wk, n, st)),
        (2 * rows + 3 * arrays, lib.sig_backward_checkpointed_workspace_bytes,
         lambda n: lib.sig_backward_checkpointed(ws._h, xp, cp, gr, kp, arrays, B, L + 1, out, wk, n, st)),
    ]
    for need, stated, call in calls:
        assert need < stated(ws._h, B, L + 1)
        assert call(need - 1) == -5 and call(need) == 0
        torch.cuda.synchronize()
        errs = O.level_errors(c[few].cpu().numpy(), ref, lengths)
        assert max(errs.values()) <= FWD_TOL, errs
        if "backward" in stated.__name__:
            assert O.grad_errors(gp[few].cpu().numpy(), gref).max() <= BWD_TOL
            gp.fill_(float("nan"))


def test_code_object_from_the_disk_cache_runs(tmp_path, monkeypatch):
    """A kernel loaded from SIG_JIT_CACHE instead of compiled gives the results of the compiled one, bit for bit."""
    import torch
    monkeypatch.setenv("SIG_JIT_CACHE", str(tmp_path))
    words = random_prefix_closed_words(77, 5, 150, 4)
    X = torch.from_numpy(make_path("iid", 78, 9, 23, 5)).cuda()
    res = []
    for _ in range(2):
        ws = S.sig_wordset_build(5, words)
        ws.upload("cuda:0")
        G = torch.from_numpy(make_grad_coeffs(79, 9, ws.size)).cuda()
        c = S.sig_forward(ws, X)
        g = S.sig_backward(ws, X, c, G)
        res.append((c.cpu().numpy(), g.cpu().numpy()))
    import os
    assert len(os.listdir(tmp_path)) == 2                         # forward and backward kernel, written once
    assert np.array_equal(res[0][0], res[1][0])
    np.testing.assert_allclose(res[0][1], res[1][1], rtol=1e-5, atol=1e-6)      # atomics: order of additions
    ws2, W = build_both("words", 5, words=words)
    check_parity(ws2, W, "words", None, make_path("iid", 78, 9, 23, 5), make_grad_coeffs(79, 9, ws2.size), what="cached kernels")


@pytest.mark.parametrize("kind", ["words", "anisotropic"])
def test_prepared_kernels_are_all_that_the_calls_compile(kind, tmp_path, monkeypatch):
    """After sig_wordset_jit_prepare and sig_wordset_jit_prepare_chunks no call of that batch size compiles a kernel, long paths in
    time chunks and short ones; the checkpointed pair needs its B * C rows besides."""
    import os

    import torch
    monkeypatch.setenv("SIG_JIT_CACHE", str(tmp_path))
    d, B = (5, 6) if kind == "words" else (3, 3)
    ws, _ = build_both(kind, d, weights=(1.0, 1.25, 1.5), cutoff=4.5, words=random_prefix_closed_words(43, 5, 120, 5))
    lib = S.load_library()
    for backward in (False, True):
        assert ws.jit_prepare(backward, B) == 0 and ws.jit_prepare_chunks(backward, B) == 0
        rows = B * int(lib.sig_checkpoint_chunks(ws._h, B, 401))
        assert ws.jit_prepare(backward, rows) == 0
    files = sorted(os.listdir(tmp_path))
    for L in (400, 12):
        x = torch.from_numpy(make_path("iid", 1950 + L, B, L, d)).cuda()
        g = torch.from_numpy(make_grad_coeffs(1951, B, ws.size)).cuda()
        S.sig_backward(ws, x, S.sig_forward(ws, x), g)
        c, ck = S.sig_forward_checkpointed(ws, x)
        S.sig_backward_checkpointed(ws, x, c, g, ck)
    torch.cuda.synchronize()
    assert sorted(os.listdir(tmp_path)) == files


def test_one_point_paths_give_zero():
    import torch
    ws, W = build_both("truncated", 3, depth=3)
    X = np.random.default_rng(0).standard_normal((5, 1, 3)).astype(np.float32)
    G = make_grad_coeffs(1, 5, ws.size)
    coeffs, gp = gpu_forward_backward(ws, X, G)
    assert coeffs.shape == (5, ws.size) and np.all(coeffs == 0.0)
    assert gp.shape == (5, 1, 3) and np.all(gp == 0.0)


def test_empty_batch_is_a_noop():
    import torch
    ws, W = build_both("truncated", 3, depth=3)
    xp = torch.zeros((0, 4, 3), dtype=torch.float32, device="cuda")
    out = S.sig_forward(ws, xp)
    assert tuple(out.shape) == (0, ws.size)
    gp = S.sig_backward(ws, xp, out, out.clone())
    assert tuple(gp.shape) == (0, 4, 3)
    torch.cuda.synchronize()


def test_repeated_points_change_nothing():
    ws, W = build_both("truncated", 3, depth=4)
    X = make_path("iid", 5, 4, 12, 3)
    Xr = np.ascontiguousarray(np.insert(X, 6, X[:, 6], axis=1))
    a, _ = gpu_forward_backward(ws, X, None)
    b, _ = gpu_forward_backward(ws, Xr, None)
    assert np.array_equal(a, b)        # exp(0) = 1: the extra segment adds exact zeros


def test_forward_is_deterministic_and_outputs_fully_overwritten():
    import torch
    wl = WORKLOADS["c1"]
    ws, W = build_for_workload(wl)
    X = workload_path(wl)
    xp = torch.from_numpy(X).cuda()
    out1 = torch.full((wl.B, ws.size), float("nan"), device="cuda")
    S.sig_forward(ws, xp, out=out1)
    out2 = S.sig_forward(ws, xp)
    torch.cuda.synchronize()
    assert torch.equal(out1, out2)
    g = torch.from_numpy(make_grad_coeffs(wl.seed, wl.B, ws.size)).cuda()
    gp = torch.full((wl.B, wl.L + 1, wl.d), float("nan"), device="cuda")
    S.sig_backward(ws, xp, out1, g, out=gp)
    torch.cuda.synchronize()
    assert torch.isfinite(gp).all()


def test_gradient_against_finite_differences_of_the_oracle_forward():
    # the benchmark spec of the gradient tolerance: fp64 central differences, 1e-3 relative
    wl = WORKLOADS["c1"]
    ws, W = build_for_workload(wl)
    B = 4
    X = workload_path(wl)[:B].astype(np.float64)
    X = np.round(X * 128) / 128                      # +-2^-12 steps stay exact in fp32
    G = make_grad_coeffs(wl.seed, B, ws.size)
    _, gp = gpu_forward_backward(ws, X.astype(np.float32), G)
    h = 2.0 ** -12
    rng = np.random.default_rng(0)
    fun = lambda Y: (O.forward_dense(Y.astype(np.float32), wl.depth) * G.astype(np.float64)).sum(axis=1)
    for _ in range(6):
        V = np.sign(rng.standard_normal(X.shape))    # +-1 directions keep the perturbed points on the grid
        num = (fun(X + h * V) - fun(X - h * V)) / (2 * h)
        ana = (gp.astype(np.float64) * V).reshape(B, -1).sum(axis=1)
        scale = np.abs(gp).reshape(B, -1).sum(axis=1)
        assert np.all(np.abs(num - ana) <= 1e-3 * scale)


def test_projection_equals_gather_of_truncation():
    # a word-projected coefficient is the same number as that word's coefficient in the full truncation
    d, depth = 4, 5
    words = random_prefix_closed_words(9, d, 200, depth)
    wsp, Wp = build_both("words", d, words=words)
    wst, Wt = build_both("truncated", d, depth=depth)
    X = make_path("iid", 77, 20, 30, d)
    a, _ = gpu_forward_backward(wsp, X, None)
    b, _ = gpu_forward_backward(wst, X, None)
    index = {w: k for k, w in enumerate(Wt)}
    pick = np.array([index[w] for w in Wp])
    ref = O.forward_dense(X, depth)[:, pick]
    lengths = np.array([len(w) for w in Wp])
    assert max(O.level_errors(a, ref, lengths).values()) <= FWD_TOL
    np.testing.assert_allclose(a, b[:, pick], rtol=2e-5, atol=1e-7)
    assert np.array_equal(wsp.user_index, np.array([{w: k for k, w in enumerate(Wp)}[w] for w in words]))


# full-size workloads in the launch configuration the benchmark times; the oracle is run on a sample
# of paths (paths are independent, so a sampled path is checked exactly as in a full comparison)
FULL = {
    "c1": None,                       # all 32 paths
    "c2": [0, 1, 63, 64, 127, 128, 200, 255],
    "c3": [0, 63, 64, 127],
    "c4a": [0, 63, 64, 300, 511],
    "c4b": [0, 63, 64, 300, 511],
    "c5": [0, 63],
}


# (name, checkpointed): the benchmark times the checkpointed pair of calls where the library offers it (c3, c4a, c5)
# and the plain pair beside it
@pytest.mark.parametrize("name,checkpointed", [(n, False) for n in FULL] + [("c3", True), ("c4a", True), ("c5", True)])
def test_full_size_workloads(name, checkpointed):
    wl = WORKLOADS[name]
    ws, W = build_for_workload(wl)
    if checkpointed:
        assert S.load_library().sig_checkpoint_bytes(ws._h, wl.B, wl.L + 1) > 0
    X = workload_path(wl)
    G = make_grad_coeffs(wl.seed, wl.B, ws.size)
    if name == "c5":
        O.set_threads(2)              # the oracle's backward keeps every intermediate signature: 2.3 GB per path
    try:
        errs, gerr = check_parity(ws, W, wl.kind, wl.depth, X, G, sample=FULL[name], what=name, checkpointed=checkpointed)
    finally:
        O.set_threads(16)
    print(f"{name}: forward level errors {errs}; gradient error max {gerr.max():.3e}")
