"""Calls on either side of the lines at which the library changes its kernel, with nothing forced, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2310_16795_amd as q
from paper_2310_16795_amd import device as dev
from paper_2310_16795_amd import synth
from test_gpu_parity import _build_layer, _check_layer, _run_layer

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    if not torch.cuda.is_available():
        pytest.fail("the GPU tests need a GPU: the HIP path has no fallback")
    return "cuda:0"


@pytest.fixture(scope="module")
def ddict(gpu, oracle_dict):
    dd = dev.DeviceDict(q.qmoe_dict_from_words(oracle_dict.words), gpu)
    yield dd
    dd.close()


# The lists of the grouping inside the first product fit the LDS, next to the paper's table, up to 12032 experts for one
# token, 11986 for 32 and 7958 for 64; more experts, up to the 16384 of the layer call, take the dispatch kernel.
@pytest.mark.parametrize("E,T", [(12032, 1), (12033, 1), (16384, 1), (11986, 32), (11987, 32), (16384, 32), (7958, 64), (8192, 64),
                                 (16384, 64)])
def test_many_experts(gpu, ddict, oracle_dict, E, T):
    w = synth.WORKLOADS["switch_base128"].scaled(n_experts=E, d_model=512, d_ff=512, n_tokens=T)
    x = w.tokens()
    idx = np.resize(np.array([E - 1, 0, E // 2, E - 1, 1], dtype=np.int32), T)
    if T > 8:
        idx[7] = E  # a token without an expert
    layer = _build_layer(w, oracle_dict, gpu, order_of=ddict, experts=sorted({int(e) for e in idx if e < E}))
    print(f"{E} experts, {T} tokens", flush=True)
    y, wsout = _run_layer(layer, ddict, x, idx, gpu)
    valid = [t for t in range(T) if idx[t] < E]
    tok_off, perm = oracle.dispatch(idx, E)
    assert np.array_equal(wsout["tok_off"], tok_off) and np.array_equal(wsout["perm"][:len(valid)], perm)
    _check_layer(w, idx, x, y, wsout, valid[:12])
    assert not y[[t for t in range(T) if idx[t] >= E]].any()
