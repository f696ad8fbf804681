"""Launches of many rows: the 2-D tiled GEMM and the packed prefill chunks.

A row's arithmetic does not depend on how many rows a launch carries, so every
comparison here is exact: a product of more than 128 rows, by whichever kernel
its shape takes and by the tiled kernel with each of its output tiles, against
the same rows in launches of at most 128 (the streaming kernel), and prompts
prefilled together, in chunks of up to 2048 rows, against each prompt prefilled
alone."""
import dataclasses

import numpy as np
import pytest
import torch  # before the library: both then share one HIP runtime

import gemm_launch as G
import synth
from paper_2402_15758_amd import Session
from paper_2402_15758_amd import binding as B

pytestmark = pytest.mark.gpu


def _gemm(dtype, x, w):
    (M, K), N = x.shape, w.shape[1]
    y = np.zeros((M, N), dtype=np.float32)
    B.chimera_debug_gemm(dtype, x.ctypes.data, w.ctypes.data, M, N, K, y.ctypes.data)
    return y


# N, K: one 16-column group up to unsplit width; K below one k-block per wave,
# ragged classes (K / 32 not a multiple of 16), split K with even and odd slices;
# the tiled kernel takes (8256, 160) and (33024, 512), the streaming kernel, in
# several row blocks, the others
@pytest.mark.parametrize("N,K", [(64, 32), (64, 96), (192, 544), (320, 1024), (2048, 2048), (1088, 5504), (8256, 160),
                                 (33024, 512)])
def test_rows_keep_their_bits_in_wide_launches(N, K):
    print(f"wide gemm N={N} K={K}", flush=True)
    torch.cuda.init()
    rng = np.random.default_rng(N + K)
    x = (rng.standard_normal((256, K)).astype(np.float32).view(np.uint32) >> 16).astype(np.uint16)
    w = (rng.standard_normal((K, N)).astype(np.float32).view(np.uint32) >> 16).astype(np.uint16)
    ref = np.concatenate([_gemm(B.CHIMERA_BF16, x[:128].copy(), w), _gemm(B.CHIMERA_BF16, x[128:].copy(), w)])
    for M in (129, 200, 256):
        y = _gemm(B.CHIMERA_BF16, x[:M].copy(), w)
        assert np.array_equal(y.view(np.uint32), ref[:M].view(np.uint32)), f"M={M}"


def _tiled(x, mtiles):
    """x [rows][K] bf16 in fragment order, `mtiles` 16-row tiles."""
    rows, K = x.shape
    t = torch.zeros((mtiles * 16, K), dtype=x.dtype, device=x.device)
    t[:rows] = x
    return t.view(mtiles, 16, K // 32, 4, 8).permute(2, 0, 3, 1, 4).contiguous()


def _untiled(t, mtiles, cols, rows):
    return t.view(cols // 32, mtiles, 4, 16, 8).permute(1, 3, 0, 2, 4).reshape(mtiles * 16, cols)[:rows]


def _outputs(kind, M, N, K, seed):
    """One product's outputs by the tiled kernel, and the same rows in launches of
    at most 128 (the streaming kernel).  W is any bits: both read the same tiles."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.randn((M, K), generator=g, device="cuda").bfloat16()
    w = torch.randn(K * N, generator=g, device="cuda").bfloat16() * 0.05
    splits = G.splits_of(1, N, K)
    hd, H = 128, N // 3 // 128
    pos = torch.arange(M, dtype=torch.int32, device="cuda") * 3 % 97
    kvoff = torch.arange(M, dtype=torch.int64, device="cuda") * N
    kvoff[::7] = -1
    qrow = torch.arange(M, dtype=torch.int32, device="cuda")
    qrow[::5] = -1
    rcos, rsin = (torch.randn((97, hd // 2), generator=g, device="cuda") for _ in range(2))
    st = torch.cuda.current_stream().cuda_stream
    keep = []

    def go(tiled_kernel, r0, rows, outs):
        mt = G.mcap(rows) // 16
        xt = _tiled(x[r0:r0 + rows], mt)
        s = G.GemmShape(None, xt.data_ptr(), mt, rows, w.data_ptr(), N, K, 0, 0, splits)
        e = G.GemmEpi(kind=kind, ldo=N, o_mtiles=mt, ldq=N // 3, head_stride=hd, H=H, hd=hd)
        parts = torch.zeros((splits, rows, N), device="cuda")
        e.part = parts.data_ptr()
        cols = N // 2 if kind == G.EPI_SWIGLU else N
        out_t = torch.zeros(mt * 16 * cols, dtype=torch.bfloat16, device="cuda")
        e.out_t, e.out_f = out_t.data_ptr(), outs[0].data_ptr() + r0 * N * 4
        e.pos, e.kvoff, e.qrow = (t.data_ptr() + r0 * t.element_size() for t in (pos, kvoff, qrow))
        e.rcos, e.rsin = rcos.data_ptr(), rsin.data_ptr()
        e.qout, e.kbase, e.vbase = (o.data_ptr() for o in outs[1:4])
        keep.extend((xt, parts, out_t))
        if tiled_kernel:
            G.launch_wide(s, e, st)
        else:
            assert G.launch(1, s, e, st)
        if kind in (G.EPI_SILU, G.EPI_SWIGLU):
            outs[4][r0:r0 + rows, :cols] = _untiled(out_t, mt, cols, rows)
        elif kind == G.EPI_PARTIAL:
            one = tiled_kernel and G.wide_sums_slices(M, N, kind)
            total = parts[0].clone()
            for i in range(1, splits):  # in slice order
                total += parts[i]
            outs[0][r0:r0 + rows] = parts[0] if one else total

    res = []
    for tiled_kernel in (True, False):
        outs = [torch.zeros((M, N), device="cuda")]
        outs += [torch.zeros((M, N), dtype=torch.bfloat16, device="cuda") for _ in range(4)]
        for r0, rows in [(0, M)] if tiled_kernel else [(r, min(128, M - r)) for r in range(0, M, 128)]:
            go(tiled_kernel, r0, rows, outs)
        res.append(outs)
    torch.cuda.synchronize()
    return res


# every output tile (256x192, 256x128, 256x96, 128x128, 128x96 rows x columns)
# under every epilogue, whole rounds of the ring and ragged classes (K = 544,
# 1088: 17 k-blocks a slice), a last row block and a last run of columns in part
WIDE = [(k, M, N, K, tile) for k in (G.EPI_F32, G.EPI_SILU, G.EPI_SWIGLU, G.EPI_QKV) for M, N, K, tile in (
    (250, 33792, 512, 0), (250, 26112, 512, 1), (250, 26112, 544, 1), (520, 18432, 512, 1), (250, 18432, 512, 2),
    (250, 18432, 544, 2), (250, 16128, 512, 3), (250, 16128, 544, 3), (130, 8448, 512, 4), (130, 8448, 544, 4))]
# slices side by side (128x128, 256x128), and added in registers by one workgroup
WIDE += [(G.EPI_PARTIAL, M, 4096, K, tile) for K in (1024, 1088) for M, tile in ((250, 3), (1000, 1), (1300, 1))]
WIDE += [(k, 1300, 4096, K, 1) for k in (G.EPI_F32, G.EPI_SILU) for K in (1024, 1088)]


@pytest.mark.parametrize("kind,M,N,K,tile", WIDE)
def test_every_tile_of_the_wide_kernel_keeps_the_rows_bits(kind, M, N, K, tile):
    print(f"wide tile {tile} kind={kind} M={M} N={N} K={K}", flush=True)
    assert G.wide_tile(M, N, K) == tile
    got, want = _outputs(kind, M, N, K, seed=M + N + K)
    assert any(bool(w.any()) for w in want)
    for a, b in zip(got, want):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))


# split reductions of a few rows (slices side by side in one workgroup): two,
# four and eight slices, ragged classes, the activation rows from one piece to
# the largest staging (7 rows of 8192 bf16), and one row more than fits
@pytest.mark.parametrize("dtype,N,K,Ms", [
    ("bf16", 192, 1024, (1, 16)), ("bf16", 64, 4096, (1, 3, 15)), ("bf16", 4096, 8192, (1, 7, 8)),
    ("bf16", 1088, 5504, (2, 11)), ("f32", 256, 768, (1, 7, 16)), ("f32", 64, 2048, (1, 15, 16)),
    ("bf16", 3584, 4096, (1, 3, 15)), ("f32", 3584, 2048, (1, 15)),  # eight slices in one workgroup
])
def test_rows_keep_their_bits_in_launches_of_a_few_rows(dtype, N, K, Ms):
    print(f"few rows {dtype} N={N} K={K}", flush=True)
    torch.cuda.init()
    rng = np.random.default_rng(N + K)
    x = rng.standard_normal((32, K)).astype(np.float32)
    w = rng.standard_normal((K, N)).astype(np.float32)
    dt = B.CHIMERA_F32
    if dtype == "bf16":
        x, w = ((v.view(np.uint32) >> 16).astype(np.uint16) for v in (x, w))
        dt = B.CHIMERA_BF16
    ref = _gemm(dt, x, w)  # 32 rows: the streaming kernel and its finishing pass
    for M in Ms:
        y = _gemm(dt, x[:M].copy(), w)
        assert np.array_equal(y.view(np.uint32), ref[:M].view(np.uint32)), f"M={M}"


# the static-scratch product stages its operands 16 bytes at a time where both
# start on a 16-byte boundary, and element by element where one does not; k-block
# counts around the four a workgroup packs, rows around the 16-row tile
@pytest.mark.parametrize("dtype,M,N,K", [("bf16", 1, 64, 32), ("bf16", 17, 192, 160), ("bf16", 130, 64, 128),
                                         ("f32", 5, 128, 16), ("f32", 16, 64, 80)])
@pytest.mark.parametrize("shift", [0, 1])
def test_static_gemm_stages_any_alignment(dtype, M, N, K, shift):
    print(f"static gemm {dtype} M={M} N={N} K={K} shift={shift}", flush=True)
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    dt = B.CHIMERA_F32 if dtype == "f32" else B.CHIMERA_BF16
    g = torch.Generator().manual_seed(M + N + K)
    x = torch.randn((M, K), generator=g).to(tdt)
    w = torch.randn((K, N), generator=g).to(tdt)
    dx = torch.zeros(M * K + shift, dtype=tdt, device="cuda")[shift:].copy_(x.view(-1))
    dw = torch.zeros(K * N + shift, dtype=tdt, device="cuda")[shift:].copy_(w.view(-1))
    y = torch.zeros((M, N), dtype=torch.float32, device="cuda")
    B.chimera_gemm_static(dt, dx.data_ptr(), dw.data_ptr(), M, N, K, y.data_ptr(),
                          torch.cuda.current_stream().cuda_stream)
    bits = (lambda t: t.numpy()) if dtype == "f32" else (lambda t: t.view(torch.int16).numpy().view(np.uint16))
    want = _gemm(dt, bits(x).copy(), bits(w).copy())
    assert np.array_equal(y.cpu().numpy().view(np.uint32), want.view(np.uint32))


# y may start at any float, on every route: a few rows with their slices in one
# workgroup, the streaming kernel unsplit and with its finishing pass, the tiled one
@pytest.mark.parametrize("dtype,M,N,K", [("bf16", 16, 64, 1024), ("bf16", 40, 8192, 64), ("f32", 40, 64, 1024),
                                         ("bf16", 129, 8256, 160)])
@pytest.mark.parametrize("shift", [1, 2, 3])
def test_static_gemm_stores_from_any_float(dtype, M, N, K, shift):
    print(f"static gemm y {dtype} M={M} N={N} K={K} shift={shift}", flush=True)
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    dt = B.CHIMERA_F32 if dtype == "f32" else B.CHIMERA_BF16
    g = torch.Generator().manual_seed(M + N + K)
    x = torch.randn((M, K), generator=g).to(tdt).cuda()
    w = torch.randn((K, N), generator=g).to(tdt).cuda()
    want = torch.zeros((M, N), dtype=torch.float32, device="cuda")
    buf = torch.full((M * N + 8,), 7.0, dtype=torch.float32, device="cuda")
    for y in (want.data_ptr(), buf.data_ptr() + 4 * shift):
        B.chimera_gemm_static(dt, x.data_ptr(), w.data_ptr(), M, N, K, y, torch.cuda.current_stream().cuda_stream)
    assert torch.equal(buf[shift:shift + M * N].view(torch.int32), want.view(-1).view(torch.int32))
    assert bool((buf[:shift] == 7).all()) and bool((buf[shift + M * N:] == 7).all())


def _states(sess):
    """What two steps after the prefill show of every sequence."""
    out = [[] for _ in range(sess.batch)]
    for _ in range(2):
        toks, n, path = sess.step()
        logits = sess.debug(B.DBG_VERIFY_LOGITS).reshape(sess.batch, sess.n_nodes, -1).view(np.uint32)
        tree = sess.debug(B.DBG_TREE_TOKENS)
        for b, o in enumerate(out):
            o += [toks[b], n[b], path[b], logits[b], tree[b]]
    return out


@pytest.mark.parametrize("model,lens", [
    ("tiny", (1, 64, 65)),
    ("tiny", (200, 17, 130)),
    ("small", (63, 129, 640)),
    ("small", (1500, 2, 900)),   # the third prompt is cut at a chunk's end
    ("small", (2049,)),          # one row past the largest chunk
    # 7B width: 129, 506, 1017 and 2033 rows together, at most 128 (256 encoder
    # rows) alone
    ("7b", (128, 1)), ("7b", (128, 127, 126, 125)), ("7b", tuple(128 - i % 3 for i in range(8))),
    ("7b", tuple(128 - i % 3 for i in range(16))),
])
def test_prompts_prefilled_together_equal_each_alone(model, lens):
    print(f"packed prefill: {model}, prompts {lens}", flush=True)
    cfg = {"tiny": synth.TINY, "small": synth.small_config(),
           "7b": dataclasses.replace(synth.LLAMA7B, n_layers=1)}[model]
    w = synth.make_weights(cfg, device="cuda", std=0.06 if cfg.d_model < 4096 else 0.02)
    prompts = [synth.make_prompt(n, cfg.vocab, 40 + i) for i, n in enumerate(lens)]
    max_len = max(lens) + 128
    every = Session(cfg, w, synth.TREE_T8, max_batch=len(lens), max_len=max_len)
    first = every.prefill(prompts)
    together = _states(every)
    for b, p in enumerate(prompts):
        one = Session(cfg, None, synth.TREE_T8, max_batch=1, max_len=max_len, share_model=every)
        assert int(one.prefill([p])[0]) == int(first[b])
        for got, want in zip(together[b], _states(one)[0]):
            assert np.array_equal(got, want)
        one.close()
    every.close()


def test_step_graph_survives_a_prefill_of_the_same_batch():
    """Requests one after another on one session, batch 2, 2, 1, 2: every
    step equals that of a session launching its kernels one by one."""
    print("graph across prefills", flush=True)
    cfg = synth.small_config()
    w = synth.make_weights(cfg, device="cuda", std=0.06)
    with torch.cuda.stream(torch.cuda.Stream()):
        graph = Session(cfg, w, synth.TREE_T32, max_batch=2, max_len=256)
        eager = Session(cfg, None, synth.TREE_T32, max_batch=2, max_len=256, share_model=graph)
        eager.set_graph(False)
        for r, lens in enumerate([(40, 77), (77, 9), (50,), (33, 64)]):
            prompts = [synth.make_prompt(n, cfg.vocab, 10 * r + i) for i, n in enumerate(lens)]
            assert np.array_equal(graph.prefill(prompts), eager.prefill(prompts))
            for got, want in zip(_states(graph), _states(eager)):
                assert all(np.array_equal(a, b) for a, b in zip(got, want))
        graph.close()
        eager.close()


def test_a_context_without_a_draft_holds_no_draft_rows():
    """A one-node context fills no draft memory in a prefill: of the chunk's
    draft rows (2048 trigram inputs and hidden rows, 4096 encoder inputs in
    float32 and storage type with their descriptors) it holds those of a step."""
    print("context bytes", flush=True)
    cfg = synth.small_config()
    w = synth.make_weights(cfg, device="cuda")
    draft = Session(cfg, w, synth.TREE_T8, max_batch=1, max_len=4096)
    plain = Session(cfg, None, (), max_batch=1, max_len=4096, share_model=draft)
    d, step = cfg.d_model, 128
    chunk = (2048 - step) * 4 * d * 2 + (4096 - step) * (d * (4 + 2) + 4 + 8 + 4)
    assert draft.ctx_arena.numel() - plain.ctx_arena.numel() >= chunk
    prompt = synth.make_prompt(2500, cfg.vocab, 3)
    assert int(plain.prefill([prompt])[0]) == int(draft.prefill([prompt])[0])
    for s in (plain, draft):
        s.close()
