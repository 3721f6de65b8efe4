"""A batch whose pull failed, pushed after the status was read: the status no longer stops the push, and the batch has
no lists.  It is consumed without effect, as it is while the status is set."""
import numpy as np
import pytest

from oracle import ctr_oracle as O
from tests.parity_util import compare_tables, run_step, to_device

pytestmark = pytest.mark.gpu

BAD_KEY = 2 ** 64 - 1


def _batch(keys, offsets, D):
    off = np.asarray(offsets, np.uint32)
    return {"keys": np.asarray(keys, np.uint64), "offsets": off,
            "grad": np.random.default_rng(len(keys)).standard_normal((off.size - 1, D)).astype(np.float32)}


@pytest.mark.parametrize("kw", [dict(), dict(bias_correction=True)])
@pytest.mark.parametrize("bad,code", [(([21, BAD_KEY, 22], [0, 3]), "CTR_E_BADKEY"), (([31, 32, 33], [0, 3, 2, 3]), "CTR_E_INVAL"),
                                      ((range(100, 400), [0, 300]), "CTR_E_FULL")])
def test_push_of_a_failed_pull_after_its_status_was_read(bad, code, kw):
    from paper_2201_05500_amd import binding as B
    D, R = 8, 128
    gt = B.CtrTable(R, D, init_seed=3, **kw)
    ot = O.OracleTable(R, D, init_seed=3, variant=O.VAR_KINGMA if kw else O.VAR_ALG2)
    good = _batch([11, 12, 13, 11], [0, 2, 4], D)
    gd = to_device(good)
    run_step(gt, ot, gd, good)
    bd = to_device(_batch(bad[0], bad[1], D))
    for refused in (False, True):                   # the pull itself fails; it is refused behind a failed lookup
        if refused:
            assert gt.lookup_pool(0, bd["keys"][:0], bd["offsets"][1:])[0] == B.CTR_OK
        st, h, _ = gt.pull_pool(0, gd["keys"] if refused else bd["keys"], gd["offsets"] if refused else bd["offsets"])
        assert st == B.CTR_OK
        assert gt.last_status() == (B.CTR_E_INVAL if refused else getattr(B, code)) and gt.last_status() == B.CTR_OK
        with pytest.raises(RuntimeError):
            gt.batch_export(h, 3)
        grad = gd["grad"] if refused else bd["grad"]
        assert gt.push_adam(0, h, grad) == B.CTR_OK and gt.push_adam(0, h, grad) == B.CTR_E_STATE
        compare_tables(gt, ot, what="after the failed pull")
    run_step(gt, ot, gd, good, what="next step")     # and the push did not count as a step
    # a lookup that fails behind a good pull leaves its batch whole
    st, h, _ = gt.pull_pool(0, gd["keys"], gd["offsets"])
    other = torch_keys([BAD_KEY])
    noalloc = B.ctr_lookup_pool_noalloc(gt._handle, 0, other.data_ptr(), 1, gd["offsets"][:1].data_ptr(), 0, None, None, gt.stream)
    assert st == B.CTR_OK and noalloc == B.CTR_OK and gt.last_status() != B.CTR_OK
    assert gt.push_adam(0, h, gd["grad"]) == B.CTR_OK and gt.last_status() == B.CTR_OK
    assert ot.pull_pool(0, good["keys"], good["offsets"])[0] == 0 and ot.push_adam(0, good["grad"]) == 0
    compare_tables(gt, ot, what="after the failed lookup")


def torch_keys(keys):
    import torch
    return torch.from_numpy(np.asarray(keys, np.uint64).view(np.int64)).to("cuda:0")
