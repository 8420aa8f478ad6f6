"""Operands that the C ABI would misread are refused before anything is launched: a tensor that is one
element broadcast over its whole extent has three zero strides, which mcf.h reads as packed.  The check
comes before the one for device tensors, so that it is tested without a GPU."""
import pytest
import torch

import paper_2506_22169_amd as mcf

MCF_EINVAL, MCF_EUNSUPPORTED = 1, 2


def _operands(batch):
    z = lambda *s: torch.zeros(s, dtype=torch.float16)
    return {"A": z(batch, 64, 64), "B": z(batch, 64, 96), "D": z(batch, 96, 64), "F": z(batch, 64, 64), "out": z(batch, 64, 64)}


def _calls(x):
    A, B, D, F, out = (x[k] for k in ("A", "B", "D", "F", "out"))
    yield "F" not in x["broadcast"], lambda: mcf.gemm_chain(A, B, D, out=out)
    yield "F" not in x["broadcast"], lambda: mcf.softmax_gemm_chain(A, B, D, 1.0, out=out)
    yield "F" not in x["broadcast"], lambda: mcf.causal_softmax_gemm_chain(A, B, D, 1.0, out=out)
    yield True, lambda: mcf.gemm_chain3(A, B, D, F, out=out)
    yield "F" not in x["broadcast"], lambda: mcf.tune_tiles(A, B, D, out=out)
    yield True, lambda: mcf.tune_tiles3(A, B, D, F, out=out)


@pytest.mark.parametrize("batch", [1, 3])
@pytest.mark.parametrize("name", ["A", "B", "D", "F", "out"])
def test_one_element_broadcast_is_refused(name, batch):
    x = _operands(batch)
    x[name] = torch.zeros(1, 1, 1, dtype=torch.float16).expand(x[name].shape)
    x["broadcast"] = name
    for concerned, call in _calls(x):
        if concerned:
            with pytest.raises(mcf.McfError) as e:
                call()
            assert e.value.status == MCF_EUNSUPPORTED, str(e.value)


def test_other_views_get_past_the_check():
    """A broadcast batch, single rows and columns, empty tensors: host tensors get as far as the device check."""
    for batch, M, N in ((3, 64, 96), (1, 1, 96), (1, 64, 0), (0, 64, 96)):
        z = lambda *s: torch.zeros(s, dtype=torch.float16)
        A, B, D = z(1, M, 64).expand(batch, M, 64) if batch else z(0, M, 64), z(batch, 64, N), z(batch, N, 64)
        with pytest.raises(mcf.McfError) as e:
            mcf.gemm_chain(A, B, D)
        assert e.value.status == MCF_EINVAL and "device" in str(e.value)


@pytest.mark.parametrize("scale", ["0.125", 0.125, torch.tensor(0.125), 1])
@pytest.mark.parametrize("offset", [2**63, -2**70, 10**30, 0])
def test_scales_and_offsets_of_any_kind(scale, offset):
    """What float() takes is a scale and any integer an offset: such calls get as far as the device check."""
    z = lambda *s: torch.zeros(s, dtype=torch.float16)
    for call in (lambda: mcf.softmax_gemm_chain(z(1, 64, 64), z(1, 64, 96), z(1, 96, 64), scale),
                 lambda: mcf.causal_softmax_gemm_chain(z(1, 64, 64), z(1, 64, 96), z(1, 96, 64), scale, offset)):
        with pytest.raises(mcf.McfError) as e:
            call()
        assert e.value.status == MCF_EINVAL and "device" in str(e.value)
