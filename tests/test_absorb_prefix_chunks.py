"""The latent prefix of a small batch in more than 64 chunks: the plan stays within the 128 partials that the
merge takes, and steps of 65 to 128 partials agree with the oracle."""
import random

import pytest

from oracle import mla_oracle as O
from paper_2509_21081_amd import binding as T
from paper_2509_21081_amd import workloads as W
from tests import helpers as Hh


def partials(heads, batch, q_len, prefix, max_suffix):
    rows = batch * q_len * heads
    need = T.typhoon_mla_decode_workspace_bytes(T.make_dims(heads, 0.07, "bf16"), T.MODES["absorb_only"],
                                                batch, q_len, prefix, max_suffix)
    # 576 absorbed columns a row, 512 columns and an LSE a partial; the rest is a few alignment gaps
    return round((need - rows * 576 * 2) / (rows * (512 * 2 + 4)))


def test_never_more_partials_than_the_merge_takes():
    rng = random.Random(3)
    for _ in range(3000):
        batch, q_len, heads = rng.randint(1, 40), rng.randint(1, 4), rng.choice((16, 32, 48, 64, 96, 128))
        prefix, suffix = rng.randint(1, 1 << rng.randint(6, 17)), rng.choice((0, rng.randint(1, 8000), 1 << 17))
        # (the gaps make up less than a partial from 16 rows on)
        assert partials(heads, batch, q_len, prefix, suffix) <= 128, (batch, q_len, heads, prefix, suffix)


@pytest.mark.parametrize("suffix_chunk,prefix_chunk", [(64, 0), (128, 0), (1024, 0), (0, 64), (64, 64)])
def test_never_more_partials_with_overrides(suffix_chunk, prefix_chunk, tune):
    # one request x 16 heads over 24192 + 4096 tokens with suffix chunks of 64 were 159 partials, refused by the merge
    # behind stages that had run
    tune(T.TUNE_SUFFIX_CHUNK, suffix_chunk)
    tune(T.TUNE_ABSORB_PREFIX_CHUNK, prefix_chunk)
    rng = random.Random(5)
    sizes = [(1, 1, 16, 24192, 4096), (1, 1, 16, 65536, 1000), (1, 1, 64, 32768, 4096), (1, 1, 128, 16384, 4096),
             (1, 1, 128, 32768, 2048)]
    sizes += [(rng.randint(1, 8), rng.randint(1, 4), rng.choice((16, 32, 64, 128)), rng.randint(8192, 1 << 17),
               rng.choice((1, 300, 2048, 4096, 100000))) for _ in range(500)]
    for size in sizes:
        batch, q_len, heads, prefix, suffix = size
        assert partials(heads, batch, q_len, prefix, suffix) <= 128, size


# (batch, heads, prefix, suffix): one row group of 64, two groups, groups of several requests' rows, no suffix, and
# last prefix chunks of one token; the least and the most chunks that plans have
SIZES = [(1, 64, 16384, 100), (1, 32, 192 * 126 + 1, 64), (1, 96, 16385, 97), (1, 16, 192 * 126, 0), (5, 16, 16500, 300),
         (3, 16, 16385, 7)]


@pytest.mark.gpu
@pytest.mark.parametrize("batch,heads,prefix,suffix", [(1, 16, 24192, 4096), (1, 128, 16384, 4096)])
def test_suffix_chunk_override_behind_a_long_prefix(batch, heads, prefix, suffix, gpu_device, tune):
    tune(T.TUNE_SUFFIX_CHUNK, 64)
    assert partials(heads, batch, 1, prefix, suffix) <= 128
    wl = W.make_workload(W.small_spec(name="override", dtype="bf16", batch=batch, heads=heads, q_len=1, prefix_len=prefix,
                                      suffix_min=suffix, suffix_max=suffix, seed=heads))
    ref, ref_lse = O.mla_decode_definition(**wl.as_float64(), pairs=[(0, h) for h in range(0, heads, 8)])
    print(f"suffix chunks of 64 behind {prefix} x {heads}", flush=True)
    got, got_lse = Hh.run_library(wl, "absorb_only", gpu_device)
    Hh.assert_parity(got, got_lse, ref, ref_lse, "bf16", f"override/{heads}")


@pytest.mark.gpu
@pytest.mark.parametrize("batch,heads,prefix,suffix", SIZES)
def test_many_prefix_chunks(batch, heads, prefix, suffix, gpu_device):
    assert 64 < partials(heads, batch, 1, prefix, suffix) <= 128
    wl = W.make_workload(W.small_spec(name="chunks", dtype="bf16", batch=batch, heads=heads, q_len=1, prefix_len=prefix,
                                      suffix_min=suffix, suffix_max=suffix, seed=prefix))
    ref, ref_lse = O.mla_decode_definition(**wl.as_float64())
    print(f"prefix chunks {batch} x {heads} x {prefix} + {suffix}", flush=True)
    got, got_lse = Hh.run_library(wl, "absorb_only", gpu_device)
    Hh.assert_parity(got, got_lse, ref, ref_lse, "bf16", f"chunks/{batch}/{heads}/{prefix}")
