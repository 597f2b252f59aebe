"""GPU parity of the step's other launch sequences, on shapes whose default
step runs scores, selection and attention in one launch, chosen through
retro_dims.flags: the scores in a launch of their own with the selection in
front of the attention (RETRO_FLAG_SEPARATE_SCORES), and the selection in a
launch of its own after them (RETRO_FLAG_SELECT_IN_SCORES).  Same bar as the other
parity tests: scores, selections, masks, A and sequence lengths bit for bit;
outputs and log-normalisers within 2e-3 (bf16) and 1e-5 (fp32) max-abs."""
import pytest

import workloads as W
from gpu_harness import run_parity

pytestmark = pytest.mark.gpu

PATHS = {"separate-scores": 1, "select-in-scores": 2}


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_09001_amd import binding
    binding.load_library()


@pytest.fixture(params=sorted(PATHS))
def path(request):
    return request.param


def test_path_tiny_fp32(path):
    run_parity(W.config(0), W.config(0).steps, flags=PATHS[path], label=f"{path} tiny-fp32")


def test_path_llama_layer_32k_shuffled(path):
    run_parity(W.config(1), 24, page_perm_seed=4, flags=PATHS[path], label=f"{path} 32k shuffled")


def test_path_batched_serving_ragged(path):
    run_parity(W.config(2), 10, page_perm_seed=2, flags=PATHS[path],
               label=f"{path} batch16 ragged")


def test_path_short_sequences_and_partial_pages(path):
    spec = W.Spec("edge-short", batch=3, num_kv_heads=2, group=3, head_dim=64, page_size=16,
                  budget=64, window=5, steps=20, dtype="bf16", prefill=(1, 17, 40), seed=9)
    run_parity(spec, 20, page_perm_seed=3, flags=PATHS[path], label=f"{path} edge short")


# steps of three launches whose attention goes through LDS (small budgets: one and two
# row tiles a wavefront) and streamed, with both page sizes and head dimensions
@pytest.mark.parametrize("hk,G,win,budget,P,d,streamed", [
    (2, 4, 8, 64, 16, 128, False), (2, 4, 33, 64, 16, 128, False), (2, 4, 64, 256, 32, 64, False),
    (2, 8, 64, 128, 16, 128, False), (2, 1, 3, 64, 16, 128, True), (4, 8, 16, 2048, 32, 64, True)])
def test_attention_kernels_of_three_launches(hk, G, win, budget, P, d, streamed):
    from paper_2508_09001_amd import binding as B
    spec = W.Spec("edge-attend", batch=2 if not streamed else 16, num_kv_heads=hk, group=G,
                  head_dim=d, page_size=P, budget=budget, window=win, steps=6, dtype="bf16",
                  prefill=(700, 33) if not streamed else (2300, 33) * 8, seed=hk + win)
    dims = B.Dims(spec.batch, hk, G, d, P, budget, win, spec.max_pages,
                  spec.batch * spec.max_pages, B.RETRO_BF16, 0.0, 0, 1, 0)
    assert (B.retro_attend_plan(dims, True)[0] > 0) == streamed
    assert B.retro_step_launches(dims) == 3
    run_parity(spec, 6, page_perm_seed=7, flags=1, label=f"attend hk={hk} W={win} P={P} d={d}")
