"""What a context takes when it is made."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw", [
    dict(T_max=8, d=64, E=2, k=1, f=64),         # as for the compression alone
    dict(T_max=64, d=72, E=4, k=2, f=136),
    dict(T_max=1024, d=64, E=8, k=2, f=128, dtype=0),
])
def test_small_context_takes_little_memory(kw):
    """The partial sums of contraction-split tiles can be 64 MB: not where no tile can be split."""
    from gpu_common import moe, say
    kw = dict(dict(R=1, local_rank=0, dtype=moe.MOE_BF16, renormalize=1), **kw)
    moe.moe_destroy(moe.moe_create(**kw))
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    ctxs = [moe.moe_create(**kw) for _ in range(4)]
    taken = (before - torch.cuda.mem_get_info()[0]) / 4
    say(f"[context] {kw}: {taken / 2**20:.1f} MiB")
    for c in ctxs:
        moe.moe_destroy(c)
    assert taken < 8 * 2**20
