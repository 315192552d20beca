"""What the Python binding keeps between calls: fault words filled in batches must not carry a caller's modes or stream
to the next one."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _draft_inputs(bad=False):
    z = torch.randn(3, 700, device="cuda")
    if bad:
        z[1, 5] = float("inf")
    return (torch.tensor([0, 3], dtype=torch.int32, device="cuda"), z, torch.zeros(3, dtype=torch.float64, device="cuda"),
            torch.rand(1, 4, device="cuda"))


def test_fault_words_filled_in_inference_mode_are_ordinary_tensors():
    import paper_2409_16560_amd as dsbd
    from paper_2409_16560_amd import binding
    args = _draft_inputs()
    binding._fault_words.clear()
    with torch.inference_mode():
        inside = dsbd.dsbd_draft_layer(*args, 4, max_prompt_beams=3)[3]     # its word comes with a batch of others
        inside.zero_()
    outside = dsbd.dsbd_draft_layer(*args, 4, max_prompt_beams=3)[3]
    assert not outside.is_inference()
    outside.zero_()
    inside.add_(1)
    assert int(outside.item()) == 0 and outside.data_ptr() != inside.data_ptr()


def test_a_fault_word_is_cleared_on_the_stream_of_the_call():
    """The call runs on a stream that is not the current one, and the current one is busy: the word must be cleared in
    front of the call, not when the current stream gets round to it."""
    import paper_2409_16560_amd as dsbd
    from paper_2409_16560_amd import binding
    args = _draft_inputs(bad=True)
    side = torch.cuda.Stream()
    a = torch.randn(8192, 8192, device="cuda", dtype=torch.bfloat16)
    torch.cuda.synchronize()
    for _ in range(3):
        binding._fault_words.clear()
        for _ in range(40):
            a @ a
        fault = dsbd.dsbd_draft_layer(*args, 4, max_prompt_beams=3, stream=side)[3]
        side.synchronize()
        torch.cuda.synchronize()
        assert int(fault.item()) == dsbd.DSBD_FAULT_NONFINITE


def test_fault_words_are_handed_out_once():
    from paper_2409_16560_amd import binding
    dev = torch.device("cuda", torch.cuda.current_device())
    words = [binding._fault_word(dev) for _ in range(200)]
    assert len({w.data_ptr() for w in words}) == 200 and all(w.numel() == 1 for w in words)
    words[3].fill_(7)
    assert sum(int(w.item()) for w in words) == 7
