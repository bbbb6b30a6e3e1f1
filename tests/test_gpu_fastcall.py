"""The native call path against the Python path of the binding, on every entry point:
the same outputs bit for bit, and the same refusals."""
import numpy as np
import pytest

from paper_2607_09207_amd import RldaError
from paper_2607_09207_amd import inputs as I
from test_gpu_parity import handle_for, torch_cuda  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu


class Refusing:
    """Stands in for the native path and takes no call."""

    def __getattr__(self, name):
        return lambda *a: None


def both(h, fn):
    """fn() through the native path (which must take it) and through Python."""
    native, taken = h._fast, []

    class Watch:
        def __getattr__(self, name):
            def call(*a):
                r = getattr(native, name)(*a)
                taken.append(r is not None)
                return r
            return call

    h._fast = Watch()
    a = fn()
    h._fast = Refusing()
    b = fn()
    h._fast = native
    assert taken == [True]
    return a, b


@pytest.mark.parametrize("given", [False, True], ids=["own_buffers", "given_buffers"])
@pytest.mark.parametrize("kv,layout", [("bf16", "page_head_slot"), ("fp8_e4m3fn", "page_slot_head"),
                                       ("f32", "page_head_slot")])
def test_native_path_is_the_python_path(torch_cuda, kv, layout, given):
    torch = torch_cuda
    hq, hkv, d = (2, 1, 64) if kv == "f32" else (8, 2, 128)
    w = I.make_multi([40, 300, 20], [4, 2, 1], hq, hkv, d, q_dtype="f32" if kv == "f32" else "bf16", kv_dtype=kv, seed=8)
    if layout == "page_slot_head":
        w = I.to_page_slot_head(w)
    t = I.to_torch(w, "cuda")
    h = handle_for(w)
    dev = t["q"].device
    h.workspace(dev, grouped=True)
    q = t["q"][:3].contiguous()
    cache = (t["k_cache"], t["v_cache"], t["block_table"], t["seq_lens"])
    sc = dict(k_scale=t["k_scale"], v_scale=t["v_scale"])
    kw = dict(sc)
    if given:
        kw.update(out=torch.empty(q.shape, device=dev), stream=torch.cuda.current_stream(), num_pages=w.num_pages)
        kw["stream"] = kw["stream"].cuda_stream
    ws = dict(workspace=torch.zeros(h.grouped_workspace_bytes + 300, dtype=torch.uint8, device=dev)[44:]) if given else {}

    def same(fn):
        a, b = both(h, lambda: fn().clone())
        assert a.dtype == b.dtype and torch.equal(a, b)

    same(lambda: h(q, *cache, **kw, **ws))
    same(lambda: h.run_noalloc(q, *cache, **kw))
    if kv != "f32":
        qs = torch.from_numpy(np.ascontiguousarray(w.q_start, np.int32)).cuda()
        mk = dict(kw, out=torch.empty(t["q"].shape, device=dev)) if given else kw
        same(lambda: h.multi(t["q"], *cache, qs, max_q_len=4, **mk, **ws))
        same(lambda: h(q, *cache, group_size=2, prefix_pages=torch.zeros(2, dtype=torch.int32, device=dev), **kw, **ws))
    new = torch.randn((3, hkv, d), device=dev).to(t["q"].dtype)
    ak = {k: v for k, v in kw.items() if k != "out"}

    def append():
        k, v = t["k_cache"].clone(), t["v_cache"].clone()
        s = {n: None if x is None else x.clone() for n, x in sc.items()}
        h.append(new, -new, k, v, t["block_table"], t["seq_lens"], **dict(ak, **s), **ws)
        return [x.view(torch.uint8) if x.element_size() == 1 else x for x in (k, v)] + [x for x in s.values() if x is not None]

    a, b = both(h, append)
    # NaN-filled slots: compared as bits
    assert all(torch.equal(x.contiguous().view(torch.uint8), y.contiguous().view(torch.uint8)) for x, y in zip(a, b))
    torch.cuda.synchronize()


def test_a_stream_object_is_taken_and_used(torch_cuda):
    torch = torch_cuda
    w = I.make_custom([40, 300, 20], 8, 2, 128, seed=18)
    t = I.to_torch(w, "cuda")
    h = handle_for(w)
    h.workspace(t["q"].device)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    fn = lambda: h(t["q"], t["k_cache"], t["v_cache"], t["block_table"], t["seq_lens"], stream=side)

    def on_side():
        o = fn()
        side.synchronize()
        return o.clone()

    a, b = both(h, on_side)
    assert torch.equal(a, b)
    # work queued on the side stream first holds the call back, work on the current one does not
    with torch.cuda.stream(side):
        torch.cuda._sleep(2_000_000)
    done = torch.cuda.Event()
    fn()
    done.record(side)
    assert not done.query()
    side.synchronize()


def test_what_the_python_checks_refuse_is_refused(torch_cuda):
    torch = torch_cuda
    w = I.make_custom([40, 300, 20], 8, 2, 128, seed=16)
    t = I.to_torch(w, "cuda")
    h = handle_for(w)
    q, k, v, bt, sl = t["q"], t["k_cache"], t["v_cache"], t["block_table"], t["seq_lens"]
    h.workspace(q.device)
    cases = [(q.float(), k, v, bt, sl), (q[:2], k, v, bt, sl), (q, k[:, :1], v, bt, sl), (q, k, v.float(), bt, sl),
             (q, k, v, bt.long(), sl), (q, k, v, bt, sl[:2]), (q, k.transpose(1, 2).contiguous().transpose(1, 2), v, bt, sl),
             (q, k.cpu(), v, bt, sl), (q, k, None, bt, sl)]
    for a in cases:
        with pytest.raises(RldaError) as e:
            h(*a)
        assert e.value.status == -1
    with pytest.raises(RldaError):
        h(q, k, v, bt, sl, num_pages=k.shape[0] + 1)
    i32 = lambda n: torch.zeros(n, dtype=torch.int32, device="cuda")
    qs = torch.arange(4, dtype=torch.int32, device="cuda")
    new = torch.zeros((3, 2, 128), dtype=q.dtype, device="cuda")
    h.workspace(q.device, grouped=True)
    for call in (lambda: h(q, k, v, bt, sl, group_size=2, prefix_pages=i32(1)),            # two groups
                 lambda: h(q, k, v, bt, sl, group_size=2, prefix_pages=i32(2).long()),
                 lambda: h(q, k, v, bt, sl, group_size=2),
                 lambda: h(q, k, v, bt, sl, group_size=0, prefix_pages=i32(2)),
                 lambda: h.multi(q, k, v, bt, sl, qs.long()),
                 lambda: h.multi(q, k, v, bt, sl, qs[:3]),
                 lambda: h.multi(q.float(), k, v, bt, sl, qs),
                 lambda: h.append(new, new[:, :1], k, v, bt, sl),
                 lambda: h.append(new.float(), new, k, v, bt, sl),
                 lambda: h.append(new, new, k, v, bt[:, :1], sl),
                 lambda: h.run_noalloc(q, k, v, bt, sl, flags=i32(2)),
                 lambda: h.run_noalloc(q, k, v, bt, sl, flags=i32(1).long()),
                 lambda: h.run_noalloc(q, k, v, bt, sl, out=torch.empty(q.shape, dtype=q.dtype, device="cuda"))):
        with pytest.raises(RldaError) as e:
            call()
        assert e.value.status == -1
    with pytest.raises(RldaError) as e:   # too small a workspace: the library's own check
        h(q, k, v, bt, sl, workspace=torch.zeros(512, dtype=torch.uint8, device="cuda"))
    assert e.value.status == -4
    torch.cuda.synchronize()
