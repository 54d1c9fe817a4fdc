"""The native marshalling of the binding's calls: well-formed calls are handled there, with the results of the Python
path behind it; a call that the library refuses still raises."""
import pytest
import torch

from paper_2104_08378_amd import sp24

pytestmark = pytest.mark.gpu


class Declines:
    """Stands in for the native module and declines every call."""

    def __getattr__(self, name):
        return lambda *a: None


def bits(r):
    return [t.contiguous().view(torch.uint8) for t in (r if isinstance(r, tuple) else (r,))]


def test_native_calls_equal_the_python_path(monkeypatch):
    g = torch.Generator(device="cuda").manual_seed(3)
    W = torch.randn((64, 128), device="cuda", generator=g).half()
    B = torch.randn((48, 128), device="cuda", generator=g).half()
    W8 = (torch.randn((64, 9 * 64), device="cuda", generator=g) * 32).to(torch.int8)
    B8 = (torch.randn((40, 9 * 64), device="cuda", generator=g) * 32).to(torch.int8)
    X = torch.randn((2, 5, 6, 64), device="cuda", generator=g)
    Wc = torch.randn((64, 9 * 64), device="cuda", generator=g).half()
    scale, bias = torch.rand(64, device="cuda", generator=g) * 1e-3, torch.randn(64, device="cuda", generator=g)
    V, m = sp24.sp24_compress(W, layout="tiled")
    V8, m8 = sp24.sp24_compress(W8, layout="tiled")
    Vc, mc = sp24.sp24_compress(Wc)
    X8 = (X * 32).to(torch.int8)
    f16, i8 = torch.float16, torch.int8
    calls = [
        lambda: sp24.sp24_prune(W), lambda: sp24.sp24_prune(W.clone(), out=torch.empty((64, 160), dtype=f16, device="cuda")[:, :128]),
        lambda: sp24.sp24_prune_transposable(W), lambda: sp24.sp24_compress(W), lambda: sp24.sp24_compress(W, layout="tiled"),
        lambda: sp24.sp24_decompress(V, m, layout="tiled"), lambda: sp24.sp24_mask_apply(W, m, layout="tiled"),
        lambda: sp24.sp24_compress_masked(W, m, layout="tiled"),
        lambda: sp24.sp24_spmm(V, m, B, torch.float32, layout="tiled"), lambda: sp24.sp24_spmm(V, m, B.t().contiguous(), f16, "n", "tiled"),
        lambda: sp24.sp24_gemm_dense(W, B, f16), lambda: sp24.sp24_spmm_splitk(V, m, B, f16, layout="tiled"),
        lambda: sp24.sp24_gemm_dense_splitk(W, B, torch.float32),
        lambda: sp24.sp24_spmm_i8_scaled(V8, m8, B8, i8, scale, 0.5, bias=bias, relu=True, inv_y_scale=3, layout="tiled"),
        lambda: sp24.sp24_gemm_dense_i8_scaled(W8, B8, f16, scale, 0.5),
        lambda: sp24.sp24_spmm_conv2d(Vc, mc, X.half(), f16, 3, 3, pad=(1, 1)), lambda: sp24.sp24_conv2d_dense(Wc, X.half(), f16, 3, 3, stride=(2, 1)),
        lambda: sp24.sp24_spmm_conv2d_i8_scaled(V8, m8, X8, i8, 3, 3, scale, 0.5, bias=bias, pad=(1, 1), layout="tiled"),
        lambda: sp24.sp24_conv2d_dense_i8_scaled(W8, X8, torch.bfloat16, 3, 3, scale, 0.5, relu=True),
    ]
    native = sp24._host

    class Counts:
        handled = 0

        def __getattr__(self, name):
            def call(*a):
                r = getattr(native, name)(*a)
                Counts.handled += r is not None
                return r
            return call

    monkeypatch.setattr(sp24, "_host", Counts())
    got = [c() for c in calls]
    assert Counts.handled == len(calls)
    monkeypatch.setattr(sp24, "_host", Declines())
    for i, (r, c) in enumerate(zip(got, calls)):
        assert all(torch.equal(x, y) for x, y in zip(bits(r), bits(c()))), i


def test_refused_calls_raise():
    W = torch.zeros((32, 64), dtype=torch.float16, device="cuda")
    V, m = sp24.sp24_compress(W)
    with pytest.raises(sp24.Sp24Error):
        sp24.sp24_prune(W.view(-1)[1:1 + 32 * 32].view(32, 32))         # not 16-byte aligned
    with pytest.raises(sp24.Sp24Error):
        sp24.sp24_spmm(V, m, W, torch.int32)                             # no such output type for float inputs
    with pytest.raises(ValueError):
        sp24.sp24_spmm(V, m, W, torch.float32, b_order="x")
    with pytest.raises(KeyError):
        sp24.sp24_spmm(V, m, W, torch.float32, layout="other")
    with pytest.raises(ValueError):
        sp24.sp24_prune(W.cpu())


def test_a_launch_error_is_raised():
    """An error that the HIP runtime holds from an earlier call comes out of the next launch as SP24_ERR_LAUNCH: it is
    raised, and the call is not made a second time."""
    W = torch.randn((64, 128), device="cuda").half()
    P, want = torch.empty_like(W), sp24.sp24_prune(W)
    V, m = sp24.sp24_compress(W)
    torch.cuda.synchronize()
    for call in (lambda: sp24.sp24_prune(W, out=P), lambda: sp24.sp24_decompress(V, m, out=P)):
        assert sp24.lib().hipSetDevice(1 << 20) != 0             # no such device: refused by the host, the current one stays
        with pytest.raises(sp24.Sp24Error) as e:
            call()
        assert e.value.status == 6                               # SP24_ERR_LAUNCH
    assert torch.equal(sp24.sp24_prune(W, out=P), want)          # and it was reported once


@pytest.mark.parametrize("pad,stride", [((1 << 70, 0), (1, 1)), ((0, -(1 << 70)), (1, 1)), ((0, 0), (1 << 70, 1)),
                                        ((0, 0), (1, 1 << 33)), ((-1, 0), (1, 1)), ((0, 0), (0, 1))])
def test_geometry_out_of_range_raises_as_the_python_path_does(monkeypatch, pad, stride):
    W = torch.zeros((32, 9 * 16), dtype=torch.float16, device="cuda")
    X = torch.zeros((1, 4, 4, 16), dtype=torch.float16, device="cuda")
    V, m = sp24.sp24_compress(W)
    raised = []
    for host in (sp24._host, Declines()):
        monkeypatch.setattr(sp24, "_host", host)
        for call in (lambda: sp24.sp24_spmm_conv2d(V, m, X, torch.float16, 3, 3, pad, stride), lambda: sp24.sp24_conv2d_dense(W, X, torch.float16, 3, 3, pad, stride)):
            with pytest.raises(Exception) as e:
                call()
            raised.append(e.type)
    assert raised[:2] == raised[2:]
