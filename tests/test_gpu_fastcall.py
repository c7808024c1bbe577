"""Device calls through the extension module _fastcall and through the Python code of binding.py: the same results bit for bit, on
torch's current stream whichever it is, and for arguments that are refused the same errors."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

HIGH = {"g128": (256, 128, 512), "g64": (256, 64, 512), "cb": (256, 128, 2048), "cbk": (256, 128, 2048), "cb8": (128, 128, 1024), "cb2": (512, 128, 4096)}


def chunks(layout, M, K, seed):
    import torch
    high, cols, head = HIGH[layout]
    r = np.random.default_rng(seed)
    c = r.integers(0, 256, (-(-M // high), K // cols, head + cols * 128), dtype=np.uint8)
    c[:, :, :head] = r.uniform(0.005, 0.02, c.shape[:2] + (head // 2,)).astype(np.float16).view(np.uint8)
    return torch.from_numpy(c.reshape(-1)).cuda()


def calls(layout, rows, half):
    """(name, call on fresh outputs -> outputs) of every entry point of the layout."""
    import torch
    import paper_2511_04477_amd as spqt
    M, K = 512, 1152
    w, ws = chunks(layout, M, K, 5), spqt.new_workspace(M, K, 4)
    x = torch.from_numpy(np.random.default_rng(6).standard_normal((rows, K)).astype(np.float16)).cuda()
    x = x if rows > 1 else x[0].contiguous()
    group = {"group": 64 if layout == "g64" else 128} if layout[0] == "g" else {}
    stem = "" if layout[0] == "g" else layout + "_"

    def gathered(masked=False):
        idx = torch.zeros(K, dtype=torch.int32, device="cuda")
        cnt = torch.zeros(1, dtype=torch.int32, device="cuda")
        if masked:
            xm = torch.zeros_like(x)
            spqt.spqt_gather_rows(x, 0.7, idx, cnt, xm)
            return idx, cnt, xm
        spqt.spqt_gather(x, 0.7, idx, cnt)
        return idx, cnt

    def new_y():
        return torch.full((rows, M) if rows > 1 else (M,), 7.0, dtype=torch.float16 if half else torch.float32, device="cuda")

    def gemv(mode, **more):
        y = new_y()
        idx, cnt = gathered() if mode == "list" else (None, None)
        name = "spqt_%sgemv" % stem + ("_rows" if layout in ("cb8", "cb2") and rows > 1 else "")
        getattr(spqt, name)(w, M, K, x, idx, cnt, y, ws, **group, **more)
        return (y,)

    def fused(own=None):
        y = new_y()
        if own is None:
            getattr(spqt, "spqt_%sgemv_fused" % stem)(w, M, K, x, 0.7, y, ws, **group)
        else:
            spqt.spqt_gemv_fused_rows(w, M, K, x, 0.7, y, ws, own_sets=own, **group)
        return (y,)

    found = [("gather", gathered), ("gather_rows", lambda: gathered(True)), ("list", lambda: gemv("list")), ("dense", lambda: gemv("dense")),
             ("shape", lambda: gemv("list", splits=2, waves=4))]
    if rows == 1:
        found.append(("fused", fused))
    if layout[0] == "g":
        found += [("fused_rows", lambda: fused(False)), ("own_sets", lambda: fused(True))]
    return found


@pytest.mark.parametrize("half", [False, True])
@pytest.mark.parametrize("layout,rows", [("g128", 1), ("g128", 3), ("g64", 2), ("cb", 1), ("cb", 4), ("cbk", 1), ("cb8", 1), ("cb8", 2), ("cb2", 1), ("cb2", 3)])
def test_same_results(monkeypatch, layout, rows, half):
    import torch
    from paper_2511_04477_amd import binding
    todo = calls(layout, rows, half)
    fast = binding._fast
    assert fast is not None
    refused = []

    class Watched:
        def __getattr__(self, name):
            def go(*a):
                rc = getattr(fast, name)(*a)
                refused.extend([name] if rc is None else [])
                return rc
            return go

    side = torch.cuda.Stream()
    for name, call in todo:
        print(f"fastcall {layout} rows={rows} half={half} {name}", flush=True)
        monkeypatch.setattr(binding, "_fast", None)
        want = [t.clone() for t in call()]
        monkeypatch.setattr(binding, "_fast", Watched())
        for stream in (torch.cuda.current_stream(), side):
            torch.cuda.synchronize()
            with torch.cuda.stream(stream):
                got = call()
            torch.cuda.synchronize()
            assert all(torch.equal(a, b) for a, b in zip(got, want)), name
    assert not refused, refused


def test_same_refusals(monkeypatch):
    """Arguments that are no plain dense tensors of the right size and type, ints or floats, or a stream: the module leaves them alone (None).  Those that it takes
    (`taken`) and those that it leaves do what the Python code does with them: the same error, or the same outputs."""
    import torch
    import paper_2511_04477_amd as spqt
    from paper_2511_04477_amd import binding
    M, K = 512, 1024
    w, ws = chunks("g128", M, K, 8), spqt.new_workspace(M, K)
    x = torch.from_numpy(np.random.default_rng(9).standard_normal(K).astype(np.float16)).cuda()
    idx = torch.zeros(K, dtype=torch.int32, device="cuda")
    cnt = torch.zeros(1, dtype=torch.int32, device="cuda")
    y = torch.zeros(M, dtype=torch.float32, device="cuda")
    fast, stream, side = binding._fast, torch.cuda.current_stream(), torch.cuda.Stream()
    at = binding.lib().at
    gather, gemv = (x, 0.5, idx, cnt, None), (w, M, K, x, idx, cnt, y, ws, None, 128, 0, 0, 0)
    assert fast.gather(at["spqt_gather"], *gather) == 0 and fast.gemv(at["spqt_gemv_ex"], *gemv) == 0
    torch.cuda.synchronize()
    listed, outputs = (idx.clone(), cnt.clone()), (idx, cnt, y)

    def outcome(fn, args):
        """What the call raises, or the outputs that it leaves behind."""
        for t, v in zip(outputs, listed if fn is spqt.spqt_gemv else (idx.new_full((K,), -1), cnt.new_full((1,), -1))):
            t.copy_(v)
        y.fill_(7.0)
        torch.cuda.synchronize()
        try:
            fn(*args)
            torch.cuda.synchronize()
            return "done", [t.cpu().numpy().tobytes() for t in outputs]
        except Exception as e:
            torch.cuda.synchronize()
            return type(e).__name__, str(e)

    wide = torch.zeros(K, 2, dtype=torch.float16, device="cuda")[:, 0]
    for fn, f, name, args, left, taken in (
            (spqt.spqt_gather, fast.gather, "spqt_gather", gather,
             [(0, x.cpu()), (0, x.float()), (0, wide), (0, None), (1, 1), (1, "a"), (1, None), (2, idx[:100]), (2, idx.long()), (3, cnt[:0]), (4, stream), (4, side),
              (4, stream.cuda_stream), (4, 0), (0, x.to_sparse()), (0, x.view(1, 1, K))],
             [(0, x[:1000]), (0, torch.nn.Parameter(x, requires_grad=False)), (0, x.view(2, 512)), (1, float("nan")), (1, float("inf")), (4, None)]),
            (spqt.spqt_gemv, fast.gemv, "spqt_gemv_ex", gemv,
             [(0, w[:-1]), (0, w.view(-1, 2)[:, 0]), (1, M + 1), (1, 512.0), (1, True), (1, 1 << 70), (2, 0), (2, 1000), (3, x[:512]), (3, x.view(2, 512)),
              (5, None), (6, y.double()), (6, y[:100]), (8, stream), (8, side), (8, 0), (9, 32), (9, 64), (12, 1 << 40)],
             [(4, None), (7, None), (7, ws[:300]), (10, -1), (10, 65), (11, 3), (12, 2)])):
        for i, other, is_left in [(*c, True) for c in left] + [(*c, False) for c in taken]:
            changed = list(args)
            changed[i] = other
            print(f"fastcall refusals {name} argument {i} {'left' if is_left else 'taken'}", flush=True)
            monkeypatch.setattr(binding, "_fast", None)
            want = outcome(fn, changed)
            monkeypatch.setattr(binding, "_fast", fast)
            assert outcome(fn, changed) == want, (name, i, other)
            assert (f(at[name], *changed) is None) == is_left, (name, i, other)
            torch.cuda.synchronize()
