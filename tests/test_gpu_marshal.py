"""The binding's native tensor checks against its own ones: what either
accepts or refuses, and with which error, is the same."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def zpp():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2407_01614_amd import zpp as mod
    return mod


class Sub(torch.Tensor):
    pass


def outcome(call):
    try:
        return call()
    except Exception as e:  # the type and the message are what is compared
        return type(e), str(e)


def arguments():
    f = torch.zeros(64, device="cuda")
    return [f, torch.zeros(64, dtype=torch.bfloat16, device="cuda"),
            torch.zeros(64, dtype=torch.uint16, device="cuda"),
            torch.zeros(64, dtype=torch.int8, device="cuda"), torch.zeros(64, device="cpu"),
            f.double(), f[::2], f[:63], f[1:], torch.zeros(0, device="cuda"), None, 7,
            f.as_subclass(Sub), torch.nn.Parameter(f.clone()), f.reshape(8, 8),
            f.reshape(8, 8).t()]


def test_native_checks_agree(zpp, monkeypatch):
    kinds = (zpp._F32, zpp._BF16, zpp._I8, zpp._U8, zpp._BF16 | zpp._OPTIONAL)
    calls = [lambda t=t, k=k, need=need: zpp._addresses(("x",), "small", t, k, need)
             for t in arguments() for k in kinds for need in (0, 63, 64, 65, 1 << 70)]
    arrays = [lambda s=s, k=k: bytes(zpp._address_array(s, k, 64, "x", "%d small"))
              for t in arguments() for k in kinds[:4]
              for s in ([t], (arguments()[0], t), [t] * 3)]
    native = [outcome(c) for c in calls + arrays]

    class Nothing:  # the binding's own checks alone
        addresses = address_array = staticmethod(lambda *a: None)

    monkeypatch.setattr(zpp, "_marshal", Nothing)
    assert native == [outcome(c) for c in calls + arrays]
    assert sum(isinstance(o, tuple) and isinstance(o[0], int) for o in native) > 20
