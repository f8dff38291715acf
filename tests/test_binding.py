"""Arguments that do not fit each other are refused by the binding before anything is enqueued.  Tensors in host memory:
what is checked here comes in front of every use of the device."""
import pytest
import torch

import paper_2502_14477_amd as esa

T0, L_C, H, H_KV, D = 300, 4, 8, 2, 64


def tensors(d=D, h_kv=H_KV, batch=None, rows=T0 + L_C, dtype=torch.bfloat16):
    lead = () if batch is None else (batch,)
    return torch.zeros(lead + (rows, h_kv, d), dtype=dtype)


def attention_calls(q, k, v, sel_k=None, sel_v=None):
    yield lambda: esa.esa_attend_indexed(q, k, v, T0, 16, 64, None)
    yield lambda: esa.esa_attend(q, k, v, T0, 16, 64, sel_k, sel_v)
    yield lambda: esa.esa_attend_reencoded(q, k, v, T0, 16, 64, sel_k, sel_v, 4096.0, 5e5)
    yield lambda: esa.esa_attend_local(q, k, v, T0, 16, 64)
    yield lambda: esa.esa_attend_finish(q, k, v, T0, 16, 64, sel_k, sel_v)


SHAPE = r"n\[|scalar_type|\bB ==|hold the current tokens"     # the check that speaks, not some later step on host memory


@pytest.mark.parametrize("name,k,v", [
    ("caches of another head size", tensors(d=128), tensors(d=128)),
    ("token rows padded to a wider head", tensors(d=32), tensors(d=32)),
    ("caches without the queries' batch", tensors(batch=3), tensors(batch=3)),
    ("caches of another type", tensors(dtype=torch.float32), tensors(dtype=torch.float32)),
    ("values of another type", tensors(), tensors(dtype=torch.float32)),
    ("values of a shorter cache", tensors(batch=1), tensors(batch=1, rows=2 * (T0 + L_C))[:, :T0].as_strided((1, T0, H_KV, D), tensors(batch=1).stride())),
    ("values of fewer heads", tensors(batch=1), tensors(batch=1)[:, :, :1]),
])
def test_attention_refuses_caches_that_do_not_fit_the_queries(name, k, v):
    q = torch.zeros((1, L_C, H, D) if k.dim() == 4 and k.shape[0] == 1 else (L_C, H, D), dtype=torch.bfloat16)
    for call in attention_calls(q, k, v):
        with pytest.raises(AssertionError, match=SHAPE):
            call()


def test_attention_refuses_an_unbatched_cache_under_batched_queries():
    q = torch.zeros((2, L_C, H, D), dtype=torch.bfloat16)
    for call in attention_calls(q, tensors(), tensors()):
        with pytest.raises(AssertionError, match=SHAPE):
            call()


@pytest.mark.parametrize("name,sel", [
    ("of another head size", tensors(d=32, rows=5)), ("of fewer heads", tensors(h_kv=1, rows=5)),
    ("of another batch", tensors(batch=2, rows=5)), ("of another type", tensors(rows=5, dtype=torch.float32))])
def test_attention_refuses_gathered_rows_that_do_not_fit(name, sel):
    q = torch.zeros((L_C, H, D), dtype=torch.bfloat16)
    calls = list(attention_calls(q, tensors(), tensors(), sel, sel))
    for call in (calls[1], calls[2], calls[4]):
        with pytest.raises(AssertionError, match=SHAPE):
            call()


def test_gathering_refuses_caches_of_another_type():
    qc, kc = torch.zeros((1, 128), dtype=torch.bfloat16), torch.zeros((T0, 128), dtype=torch.bfloat16)
    with pytest.raises(AssertionError, match=SHAPE):
        esa.esa_score_select_gather(qc, kc, 16, 200, 32, tensors(dtype=torch.float32), tensors(dtype=torch.float32))
    with pytest.raises(AssertionError, match=SHAPE):
        esa.esa_gather_kv(tensors(), tensors(dtype=torch.float32), torch.zeros(3, dtype=torch.int32))


def test_compression_refuses_weights_that_are_no_matrix_or_of_another_type():
    x, W = torch.zeros((3, 64), dtype=torch.bfloat16), torch.zeros((64, 16, 2), dtype=torch.bfloat16)
    with pytest.raises(ValueError):
        esa.esa_compress(x, W)
    with pytest.raises(ValueError):
        esa.esa_compress_qk(x, W, x, W)
    W = torch.zeros((64, 16), dtype=torch.float32)
    with pytest.raises(AssertionError, match=SHAPE):
        esa.esa_compress(x, W)
    with pytest.raises(AssertionError, match=SHAPE):
        esa.esa_compress_qk(x, W, x, W)
