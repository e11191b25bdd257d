"""Argument checks of the decoder-layer calls that pass raw pointers (host only:
the library call is replaced by a record of its arguments)."""
from types import SimpleNamespace

import pytest
import torch

from paper_2609_04875_amd import _native as N
from paper_2609_04875_amd import decoder


class OnDevice(torch.Tensor):
    """A host tensor that says it is on the device; nobody follows its pointer here."""
    is_cuda = True


def _new(*shape, dtype=torch.bfloat16):
    return torch.zeros(*shape, dtype=dtype).as_subclass(OnDevice)


@pytest.mark.parametrize("change", [
    {}, {"k": (3, 2, 128)}, {"k": (5, 2, 64)}, {"k": (5, 128)}, {"positions": (4,)}, {"q_dtype": torch.float16},
    {"k_dtype": torch.float32}, {"positions_dtype": torch.int64}, {"view": "k"}, {"view": "q"}])
def test_rope_of_q_and_k_checks_both(change, monkeypatch):
    calls = []
    monkeypatch.setattr(N, "lib", SimpleNamespace(pgsr_rope_qk_bf16=lambda *a: calls.append(a) or 0))
    q = _new(5, 8, 128, dtype=change.get("q_dtype", torch.bfloat16))
    k = _new(*change.get("k", (5, 2, 128)), dtype=change.get("k_dtype", torch.bfloat16))
    positions = _new(*change.get("positions", (5,)), dtype=change.get("positions_dtype", torch.int32))
    if change.get("view") == "k":
        k = _new(5, 4, 128)[:, :2]                    # strided: its rows are not where the kernel looks
    if change.get("view") == "q":
        q = _new(5, 16, 128)[:, ::2]
    run = lambda: decoder.rope_qk_(q, k, positions, 5e5, stream=SimpleNamespace(cuda_stream=0))  # noqa: E731
    if change:
        with pytest.raises(ValueError):
            run()
        assert not calls
    else:
        run()
        assert calls[0][:4] == (5, 8, 2, 128) and calls[0][4:7] == (q.data_ptr(), k.data_ptr(), positions.data_ptr())
