"""The Python layer's argument checks, without a GPU: what reaches the library and
what is refused, on stand-ins for device tensors and for the library."""
import ctypes

import pytest
import torch

from paper_2609_09020_amd.decoder import Decoder, ZprDecoder


class _Tensor:
    """A contiguous tensor on GPU 0, as far as the checks read one."""

    def __init__(self, shape, dtype=torch.float32, ptr=4096):
        self.shape, self.dtype, self.ptr = torch.Size(shape), dtype, ptr
        self.device = torch.device("cuda", 0)

    def get_device(self):
        return 0

    def is_contiguous(self):
        return True

    def data_ptr(self):
        return self.ptr

    def dim(self):
        return len(self.shape)

    def numel(self):
        return self.shape.numel()


class _Library:
    def __init__(self):
        self.calls = []

    def pic_decode_run(self, *a):
        self.calls.append(a)
        return 0

    pic_zpr_decode = pic_decode_run


class _Shared:
    """The kept shapes as a thread sees them while another one, of batch 1, works:
    whatever is stored, the next read may find the other's."""

    def __set_name__(self, owner, name):
        self.name = "_" + name

    def __get__(self, obj, owner):
        return getattr(obj, self.name)

    def __set__(self, obj, value):
        setattr(obj, self.name, obj.other())


def _decoder(cls, **kw):
    d = object.__new__(cls)
    d.height, d.width, d.levels, d.max_batch, d.handle = 8, 8, 2, 4, None
    d._lib, d._ptrs = _Library(), ctypes.c_void_p * 2
    for k, v in kw.items():
        setattr(d, k, v)
    return d


def _synthesis(cls=Decoder, **kw):
    return _decoder(cls, widths=(2, 4, 3), weight_dtype="f32", out_dtype="f32", nw=20, nb=7,
                    **{"_shapes_of": (None, None, None), **kw})


def _levels(batch):
    return [_Tensor((batch, 8, 8)), _Tensor((batch, 4, 4))]


def test_run_reaches_the_library_and_refuses_wrong_level_counts():
    d = _synthesis()
    out = _Tensor((2, 3, 8, 8))
    assert d.run(_levels(2), _Tensor((20,)), _Tensor((7,)), out=out, stream=0) is out
    assert d._lib.calls[0][1] == 2
    for latents in ([], _levels(2)[:1], _levels(2) + _levels(2)):
        with pytest.raises(ValueError, match="latent levels"):
            d.run(latents, _Tensor((20,)), _Tensor((7,)), out=out, batch=2, stream=0)
    assert len(d._lib.calls) == 1


def test_layers_on_the_host_are_refused():
    d = _synthesis()
    t = [torch.zeros(1, 8, 8), torch.zeros(1, 4, 4)]
    w, b = [torch.zeros(4, 2), torch.zeros(3, 4)], [torch.zeros(4), torch.zeros(3)]
    with pytest.raises(ValueError):
        d.run_layers(t, w, b, out=torch.zeros(1, 3, 8, 8))


def test_shapes_of_another_threads_batch_do_not_pass_too_small_tensors():
    class D(Decoder):
        _shapes_of = _Shared()

        def other(self):
            return (1, [(1, 8, 8), (1, 4, 4)], (1, 3, 8, 8))

    class Z(ZprDecoder):
        _shapes_of = _Shared()

        def other(self):
            return (1, [(1, 8, 8), (1, 4, 4)])

    d = _synthesis(D)
    with pytest.raises(ValueError):
        d.run(_levels(1), _Tensor((20,)), _Tensor((7,)), out=_Tensor((1, 3, 8, 8)), batch=4, stream=0)
    z = _decoder(Z, _shapes_of=(None, None))
    with pytest.raises(ValueError):
        z.decode(_Tensor((10,), torch.int32), 77, batch=4, latents=_levels(1), status=_Tensor((1,), torch.int32), stream=0)
    assert not d._lib.calls and not z._lib.calls
