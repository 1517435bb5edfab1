"""The absorb kernel of 64-token steps where it still runs: chunks of up to 128 tokens, and longer ones in launches that
cover the chip.  Its second walk, with moving exponent references, is reached by scores that grow behind the first
step and by a first step whose keys are all masked."""
import numpy as np
import pytest

from oracle import mla_oracle as O
from paper_2509_21081_amd import binding as T
from paper_2509_21081_amd import workloads as W
from tests import helpers as Hh

pytestmark = pytest.mark.gpu


def grow(wl, chunk, gain):
    """Scales the RoPE part of every key but those of the first 64 tokens of each chunk, prefix and suffix."""
    for t in range(64, wl.spec.prefix_len, 64):
        if t % chunk:
            wl.prefix_krope[t:t + 64] *= gain
    blocks = {int(x) for row in wl.block_table for i, x in enumerate(row) if (64 * i) % chunk and int(x) >= 0}
    for x in blocks:
        wl.pool[x, :, 512:] *= gain


@pytest.mark.parametrize("heads,q_len", [(64, 1), (48, 2), (128, 1)])
@pytest.mark.parametrize("gain", [256.0, 16.0, 1.0 / 64.0])
def test_scores_far_from_the_first_step_of_a_short_chunk(gain, heads, q_len, gpu_device, tune):
    """Chunks of 128 tokens: with gain 256 every chunk of more than 64 tokens overflows, and the result is
    bit-identical to the walk with moving references alone (debug flag 0x800)."""
    tune(T.TUNE_SUFFIX_CHUNK, 128)
    tune(T.TUNE_ABSORB_PREFIX_CHUNK, 128)
    wl = W.make_workload(W.small_spec(name="growth_steps", dtype="bf16", batch=4, heads=heads, q_len=q_len, prefix_len=300,
                                      suffix_min=100, suffix_max=400, seed=93))
    grow(wl, 128, gain)
    ref, ref_lse = O.mla_decode_definition(**wl.as_float64())
    for mode in ["mixed", "absorb_only"]:
        print(f"growth behind the first step, {heads} x {q_len}, gain={gain}, {mode}", flush=True)
        got, got_lse = Hh.run_library(wl, mode, gpu_device, flags=0x1000)
        alone, alone_lse = Hh.run_library(wl, mode, gpu_device, flags=0x1800)
        # (the scaled rope part is stored exactly: the bounds are those of peaked rows at gain 1)
        Hh.assert_parity(got, got_lse, ref, ref_lse, "bf16", f"growth_steps/{gain}/{mode}", peaked=True)
        Hh.assert_parity(alone, alone_lse, ref, ref_lse, "bf16", f"growth_steps/{gain}/{mode}/moving", peaked=True)
        if gain >= 256.0:
            assert np.array_equal(got, alone) and np.array_equal(got_lse, alone_lse)


@pytest.mark.parametrize("gain", [256.0, 1.0 / 64.0])
def test_scores_far_from_the_first_step_where_the_launch_covers_the_chip(gain, gpu_device, tune):
    """Two chunks of 256 tokens for each of 128 requests x 48 heads behind a prefix: 256 workgroups of four steps each."""
    tune(T.TUNE_SUFFIX_CHUNK, 256)
    wl = W.make_workload(W.small_spec(name="growth_steps_grid", dtype="bf16", batch=128, heads=48, q_len=1, prefix_len=64,
                                      suffix_min=300, suffix_max=512, seed=94))
    grow(wl, 256, gain)
    pairs = [(b, h) for b in range(0, 128, 9) for h in (0, 15, 16, 47)]
    ref, ref_lse = O.mla_decode_definition(**wl.as_float64(), pairs=pairs)
    print(f"growth behind the first step, 256 workgroups, gain={gain}", flush=True)
    got, got_lse = Hh.run_library(wl, "mixed", gpu_device)
    alone, alone_lse = Hh.run_library(wl, "mixed", gpu_device, flags=0x800)
    Hh.assert_parity(got, got_lse, ref, ref_lse, "bf16", f"growth_steps_grid/{gain}", peaked=True)
    Hh.assert_parity(alone, alone_lse, ref, ref_lse, "bf16", f"growth_steps_grid/{gain}/moving", peaked=True)
    if gain >= 256.0:
        assert np.array_equal(got, alone) and np.array_equal(got_lse, alone_lse)


@pytest.mark.parametrize("gone", [range(0, 64), range(0, 70), range(0, 128), range(64, 100)],
                         ids=["step", "head", "chunk", "behind"])
@pytest.mark.parametrize("part", ["prefix", "suffix"])
def test_keys_that_score_minus_infinity_in_short_chunks(part, gone, gpu_device, tune):
    """Chunks of 128 and 22 tokens: masked keys drop out, also where they are the whole first step, which then
    leaves no reference for the second."""
    gone = list(gone)
    keep = [t for t in range(150) if t not in gone]
    tune(T.TUNE_SUFFIX_CHUNK, 128)
    tune(T.TUNE_ABSORB_PREFIX_CHUNK, 128)
    wl = W.make_workload(W.small_spec(name="masked_steps", dtype="bf16", batch=3, heads=64, q_len=1, prefix_len=150,
                                      suffix_min=150, suffix_max=150, seed=962))
    wl.q[..., 128] = 1.0
    a = wl.as_float64()
    if part == "prefix":
        wl.prefix_krope[gone, 0] = -float("inf")
        a["prefix_ckv"], a["prefix_krope"] = a["prefix_ckv"][keep], a["prefix_krope"][keep]
    else:
        whole = a["pool"].copy()
        for table in a["block_table"]:
            for t in gone:
                wl.pool[table[t // 64], t % 64, 512] = -float("inf")
            for i, t in enumerate(keep):
                a["pool"][table[i // 64], i % 64] = whole[table[t // 64], t % 64]
        a["suffix_lens"] = np.full(3, len(keep))
    ref, ref_lse = O.mla_decode_definition(**a, pairs=[(b, h) for b in (0, 2) for h in (0, 9, 63)])
    for mode in ("absorb_only", "mixed"):
        print(f"masked keys {gone[0]} .. {gone[-1]} of the {part}, {mode}", flush=True)
        got, got_lse = Hh.run_library(wl, mode, gpu_device, flags=0x1000)
        Hh.assert_parity(got, got_lse, ref, ref_lse, "bf16", f"masked_steps/{part}/{mode}")
