"""What a bf16 context holds on the device: the workspaces of the wide pass, and the second set of the 16-column passes (16 columns
of partial sums: 16 x 32 heads x 64 chunks x 128 floats and more) only where EASYSPEC_PAIR_PASSES asks for pairs of them."""
import pytest

import easyspec_synth as synth

pytestmark = pytest.mark.gpu


def test_second_workspace_set(monkeypatch):
    import torch
    import paper_2502_02493_amd as es
    assert torch.cuda.is_available()
    cfg = synth.model_shape("llama3_8b", n_layers=1, vocab=1024)

    def held(pairs):
        if pairs is None:
            monkeypatch.delenv("EASYSPEC_PAIR_PASSES", raising=False)
        else:
            monkeypatch.setenv("EASYSPEC_PAIR_PASSES", pairs)
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        ctx = es.easyspec_create(es.make_config(cfg, 4, 128, 6), torch.cuda.current_stream().cuda_stream)
        got = free - torch.cuda.mem_get_info()[0]
        es.easyspec_destroy(ctx)
        return got

    held("0")  # what the first context of a process leaves in the allocator
    partials = 16 * 32 * 64 * 128 * 4
    wide, none, pairs = held(None), held("0"), held("1")
    assert pairs - wide >= partials, (wide, none, pairs)
    assert pairs - none >= partials, (wide, none, pairs)
