"""The native half of the binding refuses what the decode calls always refused, before anything is allocated or launched
(no GPU needed: every refusal below comes from the arguments alone)."""
import types

import pytest
import torch

from paper_2501_15021_amd import binding as akvq


def _cache():
    c = types.SimpleNamespace(B=2, Hkv=2, G=128, T_cap=64, S_cap=64, T_len=3, W=0, fine_mask=None)
    for name in ("k_codes", "v_codes", "k_meta", "v_meta", "k_sal", "v_sal", "sal_idx", "sal_cnt"):
        setattr(c, name, torch.zeros(4, dtype=torch.int32))
    c.workspace = lambda key, nbytes: torch.zeros(nbytes, dtype=torch.uint8)
    return c


HALF, ROW = torch.zeros(2, 4, 128, dtype=torch.float16), torch.zeros(2, 2, 1, 128, dtype=torch.float16)
OUT, LSE = torch.zeros(2, 4, 128), torch.zeros(2, 4)
TABLE = torch.zeros(1, 64, dtype=torch.float16)


@pytest.mark.parametrize("q,kw,error", [
    (HALF.float(), {}, AssertionError), (HALF.transpose(0, 1), {}, AssertionError), (HALF[0], {}, ValueError),
    (HALF, dict(out=OUT.half()), AssertionError), (HALF, dict(out=OUT, flags=akvq.OUT_FP16), AssertionError),
    (HALF, dict(out=torch.zeros(4, 2, 128).transpose(0, 1)), AssertionError),
    (HALF, dict(rope=(TABLE, TABLE.float())), AssertionError), (HALF, dict(rope=(TABLE, TABLE.repeat(2, 1))), AssertionError),
    (HALF, dict(rope=(TABLE.repeat(3, 1, 1), TABLE.repeat(3, 1, 1))), AssertionError),
    (HALF, dict(rope=(TABLE, TABLE, TABLE)), ValueError), (HALF, dict(n_split="4"), TypeError),
])
def test_decode_attention_refuses(q, kw, error):
    with pytest.raises(error):
        akvq.decode_attention(_cache(), q, 1.0, **{"out": OUT, "lse": LSE, **kw})


@pytest.mark.parametrize("k,v,error", [
    (ROW.float(), ROW, AssertionError), (ROW, ROW.bfloat16(), AssertionError), (ROW[:, :1], ROW[:, :1], AssertionError),
    (ROW, ROW[:1], AssertionError), (ROW.repeat(1, 1, 2, 1), ROW.repeat(1, 1, 2, 1), AssertionError),
    (torch.zeros(2, 128, 1, 2, dtype=torch.float16).transpose(1, 3), ROW, AssertionError),
])
def test_decode_step_refuses(k, v, error):
    c = _cache()
    with pytest.raises(error):
        akvq.decode_step(c, k, v, HALF, 0.8, 1.0, out=OUT, lse=LSE)
    assert c.T_len == 3


def test_a_cache_without_its_tensors_is_an_attribute_error():
    c = _cache()
    del c.sal_cnt
    with pytest.raises(AttributeError):
        akvq.decode_attention(c, HALF, 1.0, out=OUT, lse=LSE)


# an embedding that is there but not whole is not "no embedding"
@pytest.mark.parametrize("rope,error", [((None, None), TypeError), ((None, TABLE), TypeError), ((TABLE, None), TypeError),
                                        ((), ValueError), ((TABLE,), ValueError), (7, TypeError), ([None, None], TypeError)])
def test_half_a_rotary_embedding_is_refused(rope, error):
    c = _cache()
    with pytest.raises(error):
        akvq.decode_attention(c, HALF, 1.0, out=OUT, lse=LSE, rope=rope)
    with pytest.raises(error):
        akvq.decode_step(c, ROW, ROW, HALF, 0.8, 1.0, out=OUT, lse=LSE, rope=rope)
    assert c.T_len == 3


class _Asked(Exception):
    pass


def _ask(self):
    raise _Asked


def _own(cls=akvq.Cache):
    """An object of the package's class without device memory."""
    c = cls.__new__(cls)
    c.__dict__.update(vars(_cache()), _ws={}, k_win=None, v_win=None)
    return c


def _calls(c):
    yield lambda: akvq.decode_attention(c, HALF, 1.0, out=OUT, lse=LSE, rope=(TABLE, TABLE))
    yield lambda: akvq.decode_step(c, ROW, ROW, HALF, 0.8, 1.0, out=OUT, lse=LSE)


@pytest.mark.parametrize("name", ["struct", "window_struct"])
@pytest.mark.parametrize("where", ["derived", "object", "class"])
def test_a_cache_that_describes_itself_is_asked(monkeypatch, name, where):
    c = _own(type("Derived", (akvq.Cache,), {name: _ask}) if where == "derived" else akvq.Cache)
    if where == "object":
        setattr(c, name, types.MethodType(_ask, c))
    if where == "class":
        akvq.native()
        monkeypatch.setattr(akvq.Cache, name, _ask)
    for call in _calls(c):
        with pytest.raises(_Asked):
            call()
    assert c.T_len == 3


@pytest.mark.parametrize("name,answer", [("struct", None), ("struct", 5), ("struct", b"x" * 88), ("struct", akvq.akvq_window()),
                                         ("window_struct", 5), ("window_struct", akvq.akvq_cache())])
def test_an_answer_that_is_no_description_is_refused(name, answer):
    c = _own()
    setattr(c, name, lambda: answer)
    for call in _calls(c):
        with pytest.raises(TypeError):
            call()


@pytest.mark.gpu
def test_the_description_is_what_the_library_sees():
    """A group size of 77, a window without memory: refused by the library before anything is launched."""
    c = _own()
    said = c.struct()
    said.G = 77
    c.struct = lambda: said
    for call in _calls(c):
        with pytest.raises(akvq.AkvqError, match="unsupported"):
            call()
    c = _own()
    c.window_struct = lambda: akvq.akvq_window(None, None, 64)
    for call in _calls(c):
        with pytest.raises(akvq.AkvqError, match="invalid"):
            call()
    c = _own()
    c.G = 77  # the package's own method: the attribute
    for call in _calls(c):
        with pytest.raises(akvq.AkvqError, match="unsupported"):
            call()
