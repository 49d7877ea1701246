"""The binding's native half refuses what it cannot hand to the library with the binding's own error."""
import inspect

import pytest
import torch

import paper_2603_00198_amd as strd


@pytest.mark.parametrize("name,args", [
    ("score_attn", (3,)), ("score_mamba", (3, 3, 2)), ("select_topk", (1,)), ("ssd_prefill", (3, 2, 1, 3, 3)),
    ("attn_prefill", (3, 3, 3)), ("ssd_decode_step", (2, 1, 1, 2, 2)), ("attn_decode_step", (2, 3, 3)), ("linear", (2, 2)),
    ("rmsnorm", (2, 1)), ("softplus_dt", (2,))])
def test_tensors_off_the_gpu_are_refused(name, args):
    tensors = [torch.zeros([2] * d) for d in args]
    extra = {"select_topk": (1,), "ssd_decode_step": (None, torch.zeros(2, 2, 2)), "score_attn": (torch.zeros(2, 2, 2),)}
    with pytest.raises(strd.StrdError):
        getattr(strd, name)(*tensors, *extra.get(name, ()))


def test_other_objects_and_bad_descriptors_are_refused():
    with pytest.raises(strd.StrdError):
        strd.select_topk([1.0, 2.0], 1)
    with pytest.raises((strd.StrdError, TypeError)):
        strd.compact_batch(None, torch.zeros(1, dtype=torch.int32), 1, 1)
    with pytest.raises(strd.StrdError):
        strd.select_topk_varlen(torch.zeros(1, 4), [(4, 1)])


def test_every_native_entry_is_the_one_its_call_runs(monkeypatch):
    """Each entry of the native half is behind the public function of its name."""
    names = [n for n in dir(strd.binding.host()) if not n.startswith("_") and n != "set_error"]
    assert len(names) >= 18

    class Spy:
        def __getattr__(self, name):
            return lambda *args: (name, len(args))

    monkeypatch.setattr(strd.binding, "_host", Spy())
    for name in names:
        fn = getattr(strd, name)
        required = [p for p in inspect.signature(fn).parameters.values() if p.default is p.empty]
        assert fn(*[None] * len(required)) == (name, len(inspect.signature(fn).parameters))
