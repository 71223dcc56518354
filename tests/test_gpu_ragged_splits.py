"""GPU parity of the KV splits that follow the lengths of a ragged batch: one very long entry beside tiny and empty
ones (more splits than a uniform batch would get, up to the limit), all entries empty, lengths around tile borders, and
the largest batch that is split this way.  The bar is that of the other attention tests: 1e-3 of the oracle per head
(rows of several tiles are decomposed tile by tile, the oracle decomposes them once), zeros for empty entries."""
import numpy as np
import pytest
import torch

import oracle
from paper_2605_13915_amd import synth
from gpu_util import bf16_to_dev, to_dev, rel_l2

pytestmark = pytest.mark.gpu

LENGTHS = {
    "one_long": [9000, 3],
    "borders": [63, 64, 65, 0, 1, 127, 128, 129, 2500],
    "empty": [0, 0, 0],
    "many": [int(v) for v in np.random.default_rng(3).integers(0, 1200, size=64)],
    "too_many": [int(v) for v in np.random.default_rng(4).integers(0, 700, size=65)],
}


@pytest.fixture(scope="module")
def msd():
    from paper_2605_13915_amd import binding
    binding.lib()
    return binding


def _check(o, ref, lens):
    assert np.all(np.isfinite(o))
    for b, n in enumerate(lens):
        if n == 0:
            assert np.all(o[b] == 0), b
        else:
            for h in range(o.shape[1]):
                assert rel_l2(o[b, h], ref[b, h]) <= 1e-3, (b, h)


@pytest.mark.parametrize("Hq,Hkv", [(2, 1), (12, 1), (26, 1)])   # one fragment, two, and passes of 16 heads
@pytest.mark.parametrize("mode", ["token", "channel"])
@pytest.mark.parametrize("name", list(LENGTHS))
def test_grouped_query(msd, name, mode, Hq, Hkv):
    lens = LENGTHS[name]
    B, L = len(lens), max(max(lens), 600) + 30
    if Hq > 2 and B > 20:
        B, lens = 20, lens[:20]
    q = synth.queries(11, B, Hq, 128)
    if mode == "token":
        Kc, ks, Vc, vs = synth.kv_cache_per_token(11, B, Hkv, L, 128)
        omode, gmode = oracle.PER_TOKEN, msd.MSD_PER_TOKEN
    else:
        Kc, ks, Vc, vs = synth.kv_cache_per_channel(11, B, Hkv, L, 128)
        omode, gmode = oracle.PER_CHANNEL, msd.MSD_PER_CHANNEL
    kl = np.array(lens, np.int32)
    ref = oracle.attn_decode(q, Kc, Vc, ks, vs, omode, kv_len=kl)
    out = msd.msd_attn_decode_int8kv(bf16_to_dev(q), to_dev(Kc), to_dev(Vc), to_dev(ks), to_dev(vs), gmode, kv_len=to_dev(kl))
    torch.cuda.synchronize()
    _check(out.cpu().numpy(), ref, lens)


@pytest.mark.parametrize("Hq", [3, 20, 70])   # the three wave layouts, the last with two head blocks
@pytest.mark.parametrize("name", list(LENGTHS))
def test_latent(msd, name, Hq):
    lens = [min(n, 3000) for n in LENGTHS[name]]
    if Hq > 3:
        lens = lens[:9]
    B, L = len(lens), max(max(lens), 600) + 30
    rng = np.random.default_rng(5)
    C = rng.integers(-127, 128, size=(B, L, 576)).astype(np.int8)
    sc = rng.uniform(0.005, 0.02, size=(B, L)).astype(np.float32)
    q = synth.queries(12, B, Hq, 576)
    kl = np.array(lens, np.int32)
    ref = oracle.mla_decode(q, C, sc, oracle.PER_TOKEN, 512, 0.07, kv_len=kl)
    out = msd.msd_mla_decode_int8kv(bf16_to_dev(q), to_dev(C), to_dev(sc), msd.MSD_PER_TOKEN, 0.07, kv_len=to_dev(kl))
    torch.cuda.synchronize()
    _check(out.cpu().numpy(), ref, lens)
