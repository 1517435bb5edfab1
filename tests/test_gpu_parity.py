"""GPU parity: the HIP library (through its C ABI) against the fp64 oracle, element by element, on
seeded inputs small enough for the oracle yet spanning several tiles and ragged tails."""
import numpy as np
import pytest
import torch

from oracle import mla_oracle as O
from paper_2509_21081_amd import binding as T
from paper_2509_21081_amd import workloads as W
from tests import helpers as Hh

pytestmark = pytest.mark.gpu

MODES = ["mixed", "naive_only", "absorb_only"]

# (name, kwargs for small_spec)
SMALL_CASES = {
    "ragged_h16": dict(batch=3, heads=16, q_len=1, prefix_len=100, suffix_min=0, suffix_max=150),
    "mtp_h32": dict(batch=2, heads=32, q_len=2, prefix_len=70, suffix_min=1, suffix_max=200,
                    seed=21),
    "no_prefix": dict(batch=4, heads=16, q_len=1, prefix_len=0, suffix_min=1, suffix_max=130,
                      seed=22),
    "no_suffix": dict(batch=2, heads=16, q_len=1, prefix_len=97, suffix_min=0, suffix_max=0,
                      seed=23),
    "block128_qlen3": dict(batch=2, heads=16, q_len=3, prefix_len=33, suffix_min=0, suffix_max=260,
                           block_size=128, seed=24),
    "peaked": dict(batch=2, heads=16, q_len=1, prefix_len=150, suffix_min=20, suffix_max=90,
                   seed=25, q_gain=8.0),
    "h128_many_tiles": dict(batch=5, heads=128, q_len=1, prefix_len=300, suffix_min=40,
                            suffix_max=330, seed=26),
    "batch_300": dict(batch=300, heads=16, q_len=1, prefix_len=200, suffix_min=0, suffix_max=40,
                      seed=28),
    "nothing_visible": dict(batch=6, heads=16, q_len=3, prefix_len=0, suffix_min=0, suffix_max=4,
                            seed=29),
    "one_token_prefix": dict(batch=2, heads=16, q_len=1, prefix_len=1, suffix_min=0, suffix_max=1,
                             seed=30),
    "h64_kimi_like": dict(batch=3, heads=64, q_len=1, prefix_len=160, suffix_min=10, suffix_max=140,
                          seed=31),
    "wide_batch": dict(batch=70, heads=16, q_len=1, prefix_len=130, suffix_min=0, suffix_max=70,
                       seed=27),
    # 48 query rows per request: the second 32-row query block of a workgroup is half empty
    "h48_half_block": dict(batch=3, heads=48, q_len=1, prefix_len=90, suffix_min=30,
                           suffix_max=200, seed=32),
    # 96 rows: the second workgroup of a request holds one full and one empty query block;
    # q_len = 2 puts the causal edge inside a 64-token step
    "h48_mtp_empty_block": dict(batch=3, heads=48, q_len=2, prefix_len=65, suffix_min=60,
                                suffix_max=135, seed=33),
    # suffix lengths straddling the 32/64-token tile and step boundaries, causal over 3 queries
    "h32_step_edges": dict(batch=9, heads=32, q_len=3, prefix_len=64, suffix_min=61,
                           suffix_max=69, seed=34),
    # the largest supported query length: 8 positions x 16 heads = 128 rows per request (the
    # causal edge runs through one workgroup's rows), and x 32 heads = 256 rows
    "qlen8_h16": dict(batch=3, heads=16, q_len=8, prefix_len=70, suffix_min=3, suffix_max=200,
                      seed=35),
    "qlen8_h32": dict(batch=2, heads=32, q_len=8, prefix_len=40, suffix_min=8, suffix_max=150,
                      seed=36),
    # more requests than the device-side ranking of suffix lengths handles (4096): batch order
    "batch_5000": dict(batch=5000, heads=16, q_len=1, prefix_len=64, suffix_min=0, suffix_max=20,
                       seed=37),
    # one long suffix: the per-request chunk bound is reached and chunks grow instead
    "long_suffix": dict(batch=2, heads=16, q_len=1, prefix_len=40, suffix_min=9000,
                        suffix_max=9500, seed=38),
}

_cache = {}


def _workload_and_ref(case, dtype):
    key = (case, dtype)
    if key not in _cache:
        wl = W.make_workload(W.small_spec(name=case, dtype=dtype, **SMALL_CASES[case]))
        ref = O.mla_decode_definition(**wl.as_float64())
        _cache[key] = (wl, ref)
    return _cache[key]


@pytest.mark.parametrize("flags", [0, 1], ids=["mfma", "scalar"])
@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("case", list(SMALL_CASES))
def test_small_cases(case, dtype, mode, flags, gpu_device):
    if dtype == "fp32" and flags == 1:
        pytest.skip("fp32 always runs the scalar kernels")
    wl, (ref, ref_lse) = _workload_and_ref(case, dtype)
    print(f"case={case} dtype={dtype} mode={mode} flags={flags}", flush=True)
    got, got_lse = Hh.run_library(wl, mode, gpu_device, flags=flags)
    Hh.assert_parity(got, got_lse, ref, ref_lse, dtype, f"{case}/{dtype}/{mode}",
                     logit_gain=wl.spec.q_gain)


@pytest.mark.parametrize("mode", ["mixed", "absorb_only"])
@pytest.mark.parametrize("case", ["h128_many_tiles", "mtp_h32", "h48_mtp_empty_block",
                                  "ragged_h16"])
def test_forced_small_chunks(case, mode, gpu_device, tune):
    """Token chunks of one 64-token step (32 tokens for the <= 16-row kernel's wavefront shares):
    every chunk boundary, empty chunks of short requests and the merge of many latent partials."""
    tune(T.TUNE_SUFFIX_CHUNK, 64)
    tune(T.TUNE_ABSORB_PREFIX_CHUNK, 64)
    wl, (ref, ref_lse) = _workload_and_ref(case, "bf16")
    print(f"forced chunks case={case} mode={mode}", flush=True)
    got, got_lse = Hh.run_library(wl, mode, gpu_device)
    Hh.assert_parity(got, got_lse, ref, ref_lse, "bf16", f"{case}/chunk64/{mode}",
                     logit_gain=wl.spec.q_gain)


@pytest.mark.parametrize("flags", [0, 0x10000], ids=["merge_pass", "merge_inside"])
@pytest.mark.parametrize("mode", ["mixed", "absorb_only"])
def test_many_latent_partials_small_batch(mode, flags, gpu_device):
    """One and three requests of 128 heads over a 5000-token prefix and suffixes of up to 3000
    tokens: the plan cuts the tokens into many chunks to fill the chip (tens of latent partials per
    row, some empty for the shorter suffix), which the separate merge pass folds into one before
    the up-projection -- or, with debug flag bit 16, the projection kernel merges itself."""
    for batch, seed in ((1, 61), (3, 62)):
        spec = W.small_spec(name=f"many_partials_b{batch}", dtype="bf16", batch=batch, heads=128,
                            q_len=1, prefix_len=5000, suffix_min=700, suffix_max=3000, seed=seed)
        wl = W.make_workload(spec)
        a = wl.as_float64()
        ref2, ref2_lse = Hh.oracle_absorb_all_heads_parallel(O, a)
        pairs = [(b, h) for b in range(batch) for h in (0, 77, 127)]
        ref, ref_lse = O.mla_decode_definition(**a, pairs=pairs)
        print(f"many partials batch={batch} mode={mode} flags={flags:#x}", flush=True)
        got, got_lse = Hh.run_library(wl, mode, gpu_device, flags=flags)
        Hh.assert_parity(got, got_lse, ref2, ref2_lse, "bf16", f"many_partials/{mode}/absorb-form")
        Hh.assert_parity(got, got_lse, ref, ref_lse, "bf16", f"many_partials/{mode}/definition")


@pytest.mark.parametrize("heads,batch", [(16, 8), (128, 40)])
@pytest.mark.parametrize("chunks", [2, 3, 4])
def test_chunks_of_a_suffix_cost_no_precision(chunks, heads, batch, gpu_device, tune):
    """A suffix cut into 2 to 4 chunks comes out as close to fp64 as one left whole.  The partials
    are rounded to bf16 one by one, and independent roundings weighted like the partials add up to
    the rounding of one row, so the two errors are equal but for their scatter (norms over 16384
    elements and more: below 1 %); a second rounding of the merged row adds 13 %."""
    spec = W.small_spec(name="chunks", dtype="bf16", batch=batch, heads=heads, q_len=1, prefix_len=0,
                        suffix_min=64 * chunks, suffix_max=64 * chunks, seed=610 + chunks)
    wl = W.make_workload(spec)
    sample = list(range(min(batch, 8)))
    ref, _ = O.mla_decode_absorb_all_heads(**wl.as_float64(), requests=sample)
    err = {}
    for chunk in (64 * chunks, 64):
        tune(T.TUNE_SUFFIX_CHUNK, chunk)
        print(f"precision of {chunks} chunks, {batch} x {heads}: {chunk} tokens each", flush=True)
        got, _ = Hh.run_library(wl, "mixed", gpu_device)
        err[chunk] = np.linalg.norm(got[sample] - ref[sample]) / np.linalg.norm(ref[sample])
        print(f"  error {err[chunk]:.3e}", flush=True)
    assert err[64] <= 1.04 * err[64 * chunks]


@pytest.mark.parametrize("heads,q_len", [(16, 1), (32, 1), (48, 1), (64, 1), (80, 1), (48, 3), (112, 2)])
def test_latent_rows_of_partly_filled_groups(heads, q_len, gpu_device):
    """16 to 224 query rows a request, whole row groups of a workgroup and remainders: whole rows of
    the latent partials leave through LDS, and none of a neighbour's is touched."""
    spec = W.small_spec(name="groups", dtype="bf16", batch=3, heads=heads, q_len=q_len, prefix_len=70,
                        suffix_min=1, suffix_max=150, seed=640 + heads)
    wl = W.make_workload(spec)
    ref, ref_lse = O.mla_decode_absorb_all_heads(**wl.as_float64())
    for mode in ("mixed", "absorb_only"):
        print(f"rows of partly filled groups {heads} x {q_len} {mode}", flush=True)
        got, got_lse = Hh.run_library(wl, mode, gpu_device)
        Hh.assert_parity(got, got_lse, ref, ref_lse, "bf16", f"groups/{heads}x{q_len}/{mode}")


@pytest.mark.parametrize("lo,hi", [(0, 3), (30, 34), (60, 68), (92, 100), (124, 132)])
def test_chunks_of_one_and_of_several_wavefronts(lo, hi, gpu_device, tune):
    """Up to 16 rows a request: chunks of up to 64 tokens are one wavefront's, longer ones are shared by two to
    four and merged; lengths around one to four tiles, whole and as the rest behind a chunk of 128."""
    for add in (0, 128):
        tune(T.TUNE_SUFFIX_CHUNK, 128 if add else 256)
        spec = W.small_spec(name="alone", dtype="bf16", batch=24, heads=16, q_len=1, prefix_len=0,
                            suffix_min=add + lo, suffix_max=add + hi, seed=650 + hi)
        wl = W.make_workload(spec)
        ref, ref_lse = O.mla_decode_absorb_all_heads(**wl.as_float64())
        print(f"16-row chunks of {add} + {lo} to {hi} tokens", flush=True)
        got, got_lse = Hh.run_library(wl, "mixed", gpu_device)
        Hh.assert_parity(got, got_lse, ref, ref_lse, "bf16", f"alone/{add}+{lo}")


@pytest.mark.parametrize("batch", [1, 33])
@pytest.mark.parametrize("chunks", [4, 5, 16, 17, 32, 33, 64, 70])
def test_latent_partials_of_every_merge_size(chunks, batch, gpu_device, tune):
    """4 to 70 latent partials per row (64-token chunks, forced): the merge inside the projection
    kernel and every size of the merge pass, with an empty suffix chunk among them for some
    requests; one query block per head and two."""
    tune(T.TUNE_ABSORB_PREFIX_CHUNK, 64)
    tune(T.TUNE_SUFFIX_CHUNK, 64)
    n_suffix = max(1, chunks - 64)
    spec = W.small_spec(name="merge", dtype="bf16", batch=batch, heads=16, q_len=1,
                        prefix_len=64 * (chunks - n_suffix) - 5, suffix_min=0,
                        suffix_max=64 * n_suffix, seed=700 + chunks)
    wl = W.make_workload(spec)
    pairs = [(b, h) for b in range(0, batch, 8) for h in (0, 7, 15)]
    ref, ref_lse = O.mla_decode_definition(**wl.as_float64(), pairs=pairs)
    print(f"merge of {chunks} latent partials, batch={batch}", flush=True)
    got, got_lse = Hh.run_library(wl, "absorb_only", gpu_device)
    Hh.assert_parity(got, got_lse, ref, ref_lse, "bf16", f"merge_{chunks}_{batch}")


@pytest.mark.parametrize("heads,batch,chunks", [(16, 1, 1), (16, 3, 4), (128, 2, 2), (48, 5, 4), (16, 16, 5),
                                                (16, 32, 3), (16, 33, 3), (128, 4, 6)])
@pytest.mark.parametrize("splits", [0, 1, 4, 19])
def test_merge_and_projection_in_one_launch(splits, heads, batch, chunks, gpu_device, tune):
    """16 to 528 rows, 1 to 6 latent partials beside none to 19 naive ones (16 are requested up front), on
    either side of the line from which merge and projection share a launch; some requests without a
    suffix and, without a prefix, with nothing to see at all."""
    tune(T.TUNE_PREFIX_SPLITS, splits)
    tune(T.TUNE_SUFFIX_CHUNK, 64)
    spec = W.small_spec(name="one_launch", dtype="bf16", batch=batch, heads=heads, q_len=1,
                        prefix_len=128 * splits, suffix_min=0, suffix_max=64 * chunks, seed=660 + splits)
    wl = W.make_workload(spec)
    ref, ref_lse = O.mla_decode_absorb_all_heads(**wl.as_float64())
    print(f"merge and projection {heads} x {batch}, {chunks} + {splits} partials", flush=True)
    got, got_lse = Hh.run_library(wl, "mixed", gpu_device)
    Hh.assert_parity(got, got_lse, ref, ref_lse, "bf16", f"one_launch/{heads}x{batch}/{chunks}+{splits}")


def test_projection_runs_of_four_and_three_blocks(gpu_device, tune):
    """200 requests x 128 heads in three prefix splits: the projection through the ring with one latent and
    three naive partials per row, runs of four and of three blocks of 32 queries (one round of
    workgroups), a ragged last block and requests without a suffix."""
    tune(T.TUNE_PREFIX_SPLITS, 3)
    spec = W.small_spec(name="runs_4_3", dtype="bf16", batch=200, heads=128, q_len=1, prefix_len=300,
                        suffix_min=0, suffix_max=20, seed=333)
    wl = W.make_workload(spec)
    pairs = [(b, h) for b in (0, 31, 32, 95, 96, 191, 192, 199) for h in (0, 63, 127)]
    ref, ref_lse = O.mla_decode_definition(**wl.as_float64(), pairs=pairs)
    print("projection, runs of four and three blocks", flush=True)
    got, got_lse = Hh.run_library(wl, "mixed", gpu_device)
    Hh.assert_parity(got, got_lse, ref, ref_lse, "bf16", "runs_4_3")


@pytest.mark.parametrize("batch,q_len", [(31, 1), (32, 1), (33, 1), (8, 4), (9, 4), (127, 1), (129, 1), (515, 2)])
def test_query_absorption_of_partly_filled_blocks(batch, q_len, gpu_device):
    """Queries per head around 32 (all wavefronts on the same 32), 128 (a wavefront each) and beyond 1024 (four
    blocks a workgroup with 128 heads); the rows that fill a block up are nobody's."""
    heads = 128 if batch > 500 else 16
    spec = W.small_spec(name="absorption", dtype="bf16", batch=batch, heads=heads, q_len=q_len, prefix_len=40,
                        suffix_min=q_len, suffix_max=30, seed=690 + batch)
    wl = W.make_workload(spec)
    pairs = [(b, h) for b in sorted({0, 7, batch // 2, batch - 1}) for h in (0, 7, heads - 1)]
    ref, ref_lse = O.mla_decode_definition(**wl.as_float64(), pairs=pairs)
    print(f"query absorption {heads} x {batch} x {q_len}", flush=True)
    got, got_lse = Hh.run_library(wl, "absorb_only", gpu_device)
    Hh.assert_parity(got, got_lse, ref, ref_lse, "bf16", f"absorption/{batch}x{q_len}")


@pytest.mark.parametrize("heads,batch,chunks,splits,run",
                         [(16, 257, 1, 0, 1), (16, 290, 3, 9, 1), (48, 100, 2, 16, 1), (128, 33, 4, 1, 1),
                          (128, 70, 2, 3, 2), (128, 515, 1, 1, 5), (128, 300, 4, 30, 3), (64, 56, 2, 4, 1),
                          (128, 25, 3, 4, 1), (64, 50, 4, 12, 1), (128, 509, 1, 1, 8), (128, 509, 1, 15, 8)])
def test_projection_through_the_ring(heads, batch, chunks, splits, run, gpu_device, tune):
    """Runs of one to eight blocks of 32 queries (eight: every thread has a query's weights to compute) with
    a short last block, a last run shorter than the others, one to four latent partials beside none to 30
    naive ones (runs cut short by the weights' table; 16 partials x 8 blocks fill it, and the LDS, to the
    byte), some requests without a suffix and, without a prefix, with nothing to see at all."""
    blocks, parts = -(-batch // 32), chunks + splits
    one_round = -(-blocks // max(1, 256 // heads))
    assert run == -(-one_round // -(-one_round // min(8, 128 // parts)))   # (as the host cuts them)
    tune(T.TUNE_PREFIX_SPLITS, splits)
    tune(T.TUNE_SUFFIX_CHUNK, 64)
    spec = W.small_spec(name="ring", dtype="bf16", batch=batch, heads=heads, q_len=1, prefix_len=128 * splits,
                        suffix_min=0, suffix_max=64 * chunks, seed=670 + splits)
    wl = W.make_workload(spec)
    last = (batch - 1) // 32 * 32
    pairs = [(b, h) for b in sorted({0, 1, 31, 32, last - 1, last, batch - 1}) if b < batch for h in (0, 7, heads - 1)]
    ref, ref_lse = O.mla_decode_definition(**wl.as_float64(), pairs=pairs)
    print(f"projection through the ring {heads} x {batch}, {chunks} + {splits} partials", flush=True)
    got, got_lse = Hh.run_library(wl, "mixed", gpu_device)
    Hh.assert_parity(got, got_lse, ref, ref_lse, "bf16", f"ring/{heads}x{batch}/{chunks}+{splits}")


@pytest.mark.parametrize("mode", ["mixed", "naive_only", "absorb_only"])
@pytest.mark.parametrize("batch,prefix,suffix,q_len", [(1, 1, 1, 1), (1, 31, 15, 1), (1, 33, 17, 2), (3, 300, 130, 1),
                                                       (5, 65, 33, 3), (9, 0, 100, 1), (2, 257, 0, 1)])
def test_fp32_chunks_of_few_tokens(batch, prefix, suffix, q_len, mode, gpu_device):
    """fp32, 16 to 240 rows: chunks down to 16 tokens, groups of 16 lanes without a token, numbers of
    queries that are no multiple of four, one part empty; both passes in one launch."""
    wl = W.make_workload(W.small_spec(dtype="fp32", batch=batch, heads=16, q_len=q_len, prefix_len=prefix,
                                      suffix_min=min(q_len, suffix), suffix_max=suffix, seed=950 + prefix))
    ref, ref_lse = O.mla_decode_definition(**wl.as_float64())
    print(f"fp32 few tokens {mode} {batch} x {q_len} {prefix} + {suffix}", flush=True)
    got, got_lse = Hh.run_library(wl, mode, gpu_device)
    Hh.assert_parity(got, got_lse, ref, ref_lse, "fp32", f"fp32_few/{mode}")


@pytest.mark.parametrize("mode", ["mixed", "naive_only", "absorb_only"])
@pytest.mark.parametrize("prefix,suffix,q_len", [(1, 64, 1), (63, 65, 2), (64, 1, 1), (65, 129, 3),
                                                 (200, 0, 1), (0, 130, 1)])
def test_fp32_kernels_at_the_edges_of_their_tiles(prefix, suffix, q_len, mode, gpu_device):
    """fp32: token counts one below, at and above the 64-token tiles, an empty part, the causal
    edge inside a tile; 40 requests so that one chunk holds several tiles."""
    wl = W.make_workload(W.small_spec(dtype="fp32", batch=40, heads=16, q_len=q_len,
                                      prefix_len=prefix, suffix_min=min(q_len, suffix),
                                      suffix_max=suffix, seed=900 + prefix))
    pairs = [(b, h) for b in range(0, 40, 5) for h in (0, 9, 15)]
    ref, ref_lse = O.mla_decode_definition(**wl.as_float64(), pairs=pairs)
    print(f"fp32 tiles {mode} prefix={prefix} suffix={suffix} q_len={q_len}", flush=True)
    got, got_lse = Hh.run_library(wl, mode, gpu_device)
    Hh.assert_parity(got, got_lse, ref, ref_lse, "fp32", f"fp32_tiles/{mode}")


@pytest.mark.parametrize("mode", ["mixed", "absorb_only"])
def test_fp32_shows_a_nan_beside_finite_partials(mode, gpu_device, tune):
    """fp32 is what a model's outputs are checked with: a NaN in one prefix row or one suffix row
    reaches the output and LSE of every row that sees it, whichever partial holds it and however
    many finite ones stand beside it, and no other row."""
    tune(T.TUNE_PREFIX_SPLITS, 3)
    tune(T.TUNE_ABSORB_PREFIX_CHUNK, 128)
    tune(T.TUNE_SUFFIX_CHUNK, 64)
    spec = W.small_spec(dtype="fp32", batch=3, heads=16, q_len=2, prefix_len=384, suffix_min=150,
                        suffix_max=150, seed=941)
    wl = W.make_workload(spec)
    clean, clean_lse = Hh.run_library(wl, mode, gpu_device)
    assert np.isfinite(clean).all() and np.isfinite(clean_lse).all()
    # the last token of request 1, which only its last query sees (last of three suffix chunks)
    blk, at = int(wl.block_table[1, 149 // 64]), 149 % 64
    wl.pool[blk, at, 570] = float("nan")
    print(f"fp32 NaN in a suffix row, {mode}", flush=True)
    got, got_lse = Hh.run_library(wl, mode, gpu_device)
    hit = np.zeros((3, 2), bool)
    hit[1, 1] = True
    assert np.isnan(got[hit]).all() and np.isnan(got_lse[hit]).all()
    assert np.array_equal(got[~hit], clean[~hit]) and np.array_equal(got_lse[~hit], clean_lse[~hit])
    # every part of the prefix in turn
    for t in (5, 200, 383):
        wl = W.make_workload(spec)
        wl.prefix_krope[t, 3] = float("nan")
        print(f"fp32 NaN in prefix row {t}, {mode}", flush=True)
        got, got_lse = Hh.run_library(wl, mode, gpu_device)
        assert np.isnan(got).all() and np.isnan(got_lse).all()


# tokens that are masked: one of the first, a middle and the last tile, a run longer than a tile, all
MASKED = {"first": [0], "middle": [77], "last": [149], "two": [5, 21], "run": list(range(3, 73)),
          "all": list(range(150))}


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("part", ["prefix", "suffix", "both"])
@pytest.mark.parametrize("masked", list(MASKED))
def test_fp32_drops_keys_that_score_minus_infinity(masked, part, mode, gpu_device):
    """fp32: a key masked through its RoPE part (a score of -inf) drops out like a token that is not
    there, also where it is all that a group of 16 lanes, a chunk or a row has to see.  One request
    (chunks of 16 and 32 tokens) and twenty (chunks of several tiles)."""
    for batch in (1, 20):
        spec = W.small_spec(name="masked", dtype="fp32", batch=batch, heads=16, q_len=1, prefix_len=150,
                            suffix_min=150, suffix_max=150, seed=960 + batch)
        wl = W.make_workload(spec)
        wl.q[..., 128] = 1.0
        a = wl.as_float64()
        gone = MASKED[masked]
        keep = [t for t in range(150) if t not in gone]
        if part != "suffix":
            wl.prefix_krope[gone, 0] = -float("inf")
            a["prefix_ckv"], a["prefix_krope"] = a["prefix_ckv"][keep], a["prefix_krope"][keep]
        if part != "prefix":
            bs, whole = spec.block_size, a["pool"].copy()
            for table in a["block_table"]:
                for t in gone:
                    wl.pool[table[t // bs], t % bs, 512] = -float("inf")
                for i, t in enumerate(keep):
                    a["pool"][table[i // bs], i % bs] = whole[table[t // bs], t % bs]
            a["suffix_lens"] = np.full(batch, len(keep))
        ref, ref_lse = O.mla_decode_definition(**a, pairs=[(b, h) for b in range(0, batch, 7) for h in (0, 9, 15)])
        print(f"fp32 masked keys {masked} {part} {mode} batch={batch}", flush=True)
        got, got_lse = Hh.run_library(wl, mode, gpu_device)
        Hh.assert_parity(got, got_lse, ref, ref_lse, "fp32", f"fp32_masked/{masked}/{part}/{mode}/{batch}")


@pytest.mark.parametrize("flags", [0, 0x400], ids=["pipelined", "8-wave"])
@pytest.mark.parametrize("prefix_len", [31, 32, 40, 288, 1024, 1100])
def test_pipelined_prefix_kernel_long_runs(prefix_len, flags, gpu_device, tune):
    """More than 128 queries per head select the software-pipelined prefix kernel; one split
    (forced) makes a single workgroup walk the whole prefix: a partial block only, one full
    block, full + partial, one block more than the transfer look-ahead, and long runs with and
    without a partial tail.  Also with the 8-wavefront kernel, its fallback, running alone."""
    tune(T.TUNE_PREFIX_SPLITS, 1)
    spec = W.small_spec(name=f"pipe_{prefix_len}", dtype="bf16", batch=200, heads=16, q_len=1,
                        prefix_len=prefix_len, suffix_min=0, suffix_max=40, seed=41 + prefix_len)
    wl = W.make_workload(spec)
    ref, ref_lse = O.mla_decode_definition(**wl.as_float64())
    print(f"pipelined prefix, prefix_len={prefix_len} flags={flags}", flush=True)
    got, got_lse = Hh.run_library(wl, "mixed", gpu_device, flags=flags)
    Hh.assert_parity(got, got_lse, ref, ref_lse, "bf16", f"pipe_{prefix_len}")


@pytest.mark.parametrize("gain,first", [(256.0, 64), (256.0, 1000), (16.0, 64), (1.0 / 64.0, 64)])
def test_prefix_scores_far_from_the_first_block(gain, first, gpu_device, tune):
    """The RoPE part of the keys from token `first` on is scaled by `gain` (a power of two, and
    that part of a key is stored as given, so the oracle sees exactly what the kernels see): the
    scores there lie far above (or below) those of the first block, whose maximum the pipelined
    kernel takes as its exponent reference.  With gain 256 its denominators overflow for every
    query: it must notice, form the exact maxima in a scores-only pass and walk the prefix
    again.  The 8-wavefront kernel (moving references; debug flag 0x400) is held against the
    oracle on the same inputs."""
    tune(T.TUNE_PREFIX_SPLITS, 1)
    spec = W.small_spec(name="growth", dtype="bf16", batch=150, heads=16, q_len=1,
                        prefix_len=1100, suffix_min=0, suffix_max=30, seed=77)
    wl = W.make_workload(spec)
    wl.prefix_krope[first:] *= gain
    ref, ref_lse = O.mla_decode_definition(**wl.as_float64())
    print(f"prefix score growth, gain={gain} from token {first}", flush=True)
    got, got_lse = Hh.run_library(wl, "mixed", gpu_device)
    alone, alone_lse = Hh.run_library(wl, "mixed", gpu_device, flags=0x400)
    # only the rope part of the keys was scaled, and it is stored exactly, so nothing grows with
    # the gain; but the rows are peaked, which exposes the rounding of the top logit's noPE part
    Hh.assert_parity(got, got_lse, ref, ref_lse, "bf16", f"growth_{gain}_{first}", peaked=True)
    Hh.assert_parity(alone, alone_lse, ref, ref_lse, "bf16", f"growth_{gain}_{first}/8-wave",
                     peaked=True)


@pytest.mark.parametrize("batch", [65, 96, 128])
@pytest.mark.parametrize("prefix_len,splits,gain",
                         [(1, 1, 1.0), (32, 1, 1.0), (33, 1, 1.0), (64, 1, 1.0), (95, 1, 1.0),
                          (96, 1, 1.0), (288, 1, 1.0), (600, 1, 1.0), (1100, 2, 1.0),
                          (1000, 0, 1.0), (1100, 1, 256.0)])
def test_prefix_kernel_with_wavefront_pairs(prefix_len, splits, gain, batch, gpu_device, tune):
    """65 to 128 queries per head: the two pairs of wavefronts take half of a split's blocks each.
    One block (one pair sees nothing), odd and even numbers of blocks with and without a partial
    last one, shorter and longer than the ring, several splits, and (gain) denominators that
    overflow in one pair alone, which makes the whole workgroup walk again."""
    tune(T.TUNE_PREFIX_SPLITS, splits)
    spec = W.small_spec(name="pairs", dtype="bf16", batch=batch, heads=16, q_len=1,
                        prefix_len=prefix_len, suffix_min=0, suffix_max=30, seed=500 + prefix_len)
    wl = W.make_workload(spec)
    wl.prefix_krope[700:] *= gain
    ref, ref_lse = O.mla_decode_definition(**wl.as_float64())
    print(f"paired prefix, batch={batch} prefix_len={prefix_len} splits={splits}", flush=True)
    got, got_lse = Hh.run_library(wl, "mixed", gpu_device, flags=0x20000)   # whatever the length
    Hh.assert_parity(got, got_lse, ref, ref_lse, "bf16", f"pairs_{batch}_{prefix_len}",
                     peaked=gain != 1.0)


# (queries per head, flags) of every kernel of the prefix pass: token-split, wavefront pairs, pipelined
PREFIX_KERNELS = {"token_split": (100, 0), "pairs": (100, 0x20000), "pipelined": (160, 0)}


@pytest.mark.parametrize("kernel", list(PREFIX_KERNELS))
@pytest.mark.parametrize("prefix_len", [96, 90, 64, 33, 352])
def test_prefix_kernels_with_values_that_are_not_finite(prefix_len, kernel, gpu_device, tune):
    """One split of 2, 3 or 11 blocks (odd: the pairs share the middle one), whole and partial last
    blocks.  An infinite value reaches exactly its own column; a key that scores -inf drops out
    like a token that is not there, in every block; where the wavefronts of a workgroup see
    different blocks of a query, a NaN in one of them takes the whole split with it and not a part."""
    batch, flags = PREFIX_KERNELS[kernel]
    tune(T.TUNE_PREFIX_SPLITS, 1)
    spec = W.small_spec(name="inf", dtype="bf16", batch=batch, heads=16, q_len=1,
                        prefix_len=prefix_len, suffix_min=5, suffix_max=30, seed=77 + prefix_len)
    wl = W.make_workload(spec)
    wl.q[..., 0] = 1.0
    d = wl.to(gpu_device)
    dims = Hh.dims_of(wl)

    def run(change=None):
        pk, pv = T.typhoon_mla_expand_prefix(dims, d.prefix_ckv, d.prefix_krope, d.w_uk, d.w_uv)
        if change:
            change(pk.view(torch.bfloat16), pv.view(torch.bfloat16))
        old = T.typhoon_mla_set_debug_flags(flags)
        try:
            out, lse = T.typhoon_mla_decode(
                dims, "mixed", d.q, prefix_len, prefix_k=pk, prefix_v=pv, suffix_pool=d.pool,
                block_table=d.block_table, suffix_lens=d.suffix_lens,
                max_suffix_len=wl.max_suffix_len, w_uk=d.w_uk, w_uv=d.w_uv)
            torch.cuda.synchronize(gpu_device)
        finally:
            T.typhoon_mla_set_debug_flags(old)
        return out.double().cpu().numpy(), lse.double().cpu().numpy()

    clean, clean_lse = run()
    assert np.isfinite(clean).all() and np.isfinite(clean_lse).all()
    # a token of the first, the middle and the last block
    for t in sorted({3, 32 * (((prefix_len + 31) // 32) // 2) + 5 if prefix_len > 40 else 7,
                     prefix_len - 1}):
        print(f"not finite: {kernel} prefix_len={prefix_len} token {t}", flush=True)

        def inf_value(k, v):
            v[Hh.v_offset(3, prefix_len, t, 7, "bf16")] = float("inf")
        got, got_lse = run(inf_value)
        assert np.isposinf(got[:, :, 3, 7]).all()
        got[:, :, 3, 7] = clean[:, :, 3, 7]
        assert np.array_equal(got, clean) and np.array_equal(got_lse, clean_lse)

        def masked_key(k, v):
            for h in range(16):
                k[Hh.k_offset(h, prefix_len, t, 0, "bf16")] = -float("inf")
        got, got_lse = run(masked_key)
        keep = [i for i in range(prefix_len) if i != t]
        a = wl.as_float64()
        a["prefix_ckv"], a["prefix_krope"] = a["prefix_ckv"][keep], a["prefix_krope"][keep]
        ref, ref_lse = O.mla_decode_definition(**a, pairs=[(b, h) for b in range(0, batch, 9)
                                                           for h in (0, 3, 15)])
        Hh.assert_parity(got, got_lse, ref, ref_lse, "bf16", f"masked_key_{kernel}")

        if kernel == "token_split":   # (its wavefronts' partials are weighted one by one)
            continue

        def nan_key(k, v):
            for h in range(16):
                k[Hh.k_offset(h, prefix_len, t, 0, "bf16")] = float("nan")
        # (a row whose only split scored NaN carries no prefix partial: the suffix alone is left)
        got, got_lse = run(nan_key)
        a = wl.as_float64()
        a["prefix_ckv"], a["prefix_krope"] = a["prefix_ckv"][:0], a["prefix_krope"][:0]
        ref, ref_lse = O.mla_decode_definition(**a, pairs=[(b, h) for b in range(0, batch, 9)
                                                           for h in (0, 3, 15)])
        Hh.assert_parity(got, got_lse, ref, ref_lse, "bf16", f"nan_key_{kernel}")


@pytest.mark.parametrize("heads,flags", [(16, 0), (32, 0), (64, 0), (128, 0), (128, 0x2000)])
@pytest.mark.parametrize("masked", ["first", "run", "head", "all"])
def test_absorb_kernels_drop_keys_that_score_minus_infinity(masked, heads, flags, gpu_device, tune):
    """Kernels for up to 16, 32, 64 and 128 rows (debug flag bit 13), latent prefix and suffix in one chunk
    each: keys masked through their RoPE part drop out, also where they are all that the first tokens of the chunk
    have, whose maxima the 64- and 128-row kernels (32 and 64 of them) take as references for those behind."""
    gone = list(range(70)) if masked == "head" else MASKED[masked]
    keep = [t for t in range(150) if t not in gone]
    tune(T.TUNE_SUFFIX_CHUNK, 256)
    tune(T.TUNE_ABSORB_PREFIX_CHUNK, 256)
    for part in ("prefix", "suffix"):
        spec = W.small_spec(name="masked", dtype="bf16", batch=3, heads=heads, q_len=1, prefix_len=150,
                            suffix_min=150, suffix_max=150, seed=961)
        wl = W.make_workload(spec)
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
        ref, ref_lse = O.mla_decode_definition(**a, pairs=[(b, h) for b in (0, 2) for h in (0, 9, 15)])
        for mode in ("absorb_only", "mixed"):
            print(f"masked keys {masked} of the {part}, {heads} heads, flags {flags:#x}, {mode}", flush=True)
            got, got_lse = Hh.run_library(wl, mode, gpu_device, flags=flags)
            Hh.assert_parity(got, got_lse, ref, ref_lse, "bf16", f"masked/{masked}/{part}/{heads}/{mode}")


@pytest.mark.parametrize("heads", [16, 32, 64])
@pytest.mark.parametrize("token", [5, 40, 90, 127, 150])
def test_a_nan_takes_its_whole_chunk_of_a_suffix(token, heads, gpu_device, tune):
    """Kernels for up to 16, 32 and 64 rows a request, chunks of 128 and 72 tokens: a key that scores NaN
    takes the whole chunk with it and not the part of a wavefront (up to 16 rows each of the four has
    32 of the 128 tokens), and no other chunk or request."""
    tune(T.TUNE_SUFFIX_CHUNK, 128)
    spec = W.small_spec(name="nan_chunk", dtype="bf16", batch=3, heads=heads, q_len=1, prefix_len=64,
                        suffix_min=200, suffix_max=200, seed=970)
    wl = W.make_workload(spec)
    clean, clean_lse = Hh.run_library(wl, "mixed", gpu_device)
    assert np.isfinite(clean).all() and np.isfinite(clean_lse).all()
    a = wl.as_float64()
    table = a["block_table"][1]
    wl.pool[table[token // 64], token % 64, 570] = float("nan")
    if token < 128:     # the second chunk is left, its 72 tokens in front
        whole = a["pool"].copy()
        for i in range(72):
            a["pool"][table[i // 64], i % 64] = whole[table[(128 + i) // 64], (128 + i) % 64]
    a["suffix_lens"] = np.array([200, 72 if token < 128 else 128, 200])
    ref, ref_lse = O.mla_decode_definition(**a, pairs=[(1, h) for h in range(0, heads, 5)])
    print(f"NaN at suffix token {token}, {heads} heads", flush=True)
    got, got_lse = Hh.run_library(wl, "mixed", gpu_device)
    Hh.assert_parity(got, got_lse, ref, ref_lse, "bf16", f"nan_chunk/{heads}/{token}")
    assert np.array_equal(got[[0, 2]], clean[[0, 2]]) and np.array_equal(got_lse[[0, 2]], clean_lse[[0, 2]])


@pytest.mark.parametrize("gain", [256.0, 16.0, 1.0 / 64.0])
def test_suffix_scores_far_from_the_first_step(gain, gpu_device, tune):
    """The same for the absorb pass over the suffix with more than 32 query rows per request: the
    pipelined 64-row kernel first walks a chunk with exponent references fixed at its first 32 tokens
    and walks it again with exact ones if its denominators overflowed (the kernel of 64-token steps, which
    has shorter chunks: test_absorb64_steps.py).  The RoPE part of every
    cached suffix row behind the first block is scaled (stored as given, so exact for the
    oracle); one chunk per request (forced), so with gain 256 every workgroup overflows and the
    result is bit-identical to the walk with exact references alone (debug flag 0x800)."""
    tune(T.TUNE_SUFFIX_CHUNK, 4096)
    spec = W.small_spec(name="suffix_growth", dtype="bf16", batch=6, heads=128, q_len=1,
                        prefix_len=40, suffix_min=200, suffix_max=700, seed=91)
    wl = W.make_workload(spec)
    wl.pool[:, :, 512:] *= gain
    for b in range(spec.batch):
        wl.pool[int(wl.block_table[b, 0]), :, 512:] /= gain     # the first 64 tokens stay
    ref, ref_lse = O.mla_decode_definition(**wl.as_float64())
    print(f"suffix score growth, gain={gain}", flush=True)
    # (the scaled rope part is stored exactly: the bounds are those of peaked rows at gain 1)
    for mode in ["mixed", "absorb_only"]:
        got, got_lse = Hh.run_library(wl, mode, gpu_device)
        alone, alone_lse = Hh.run_library(wl, mode, gpu_device, flags=0x800)
        Hh.assert_parity(got, got_lse, ref, ref_lse, "bf16", f"suffix_growth_{gain}/{mode}",
                         peaked=True)
        Hh.assert_parity(alone, alone_lse, ref, ref_lse, "bf16",
                         f"suffix_growth_{gain}/{mode}/moving", peaked=True)
        if gain >= 256.0 and mode == "mixed":
            assert np.array_equal(got, alone) and np.array_equal(got_lse, alone_lse)


# requests with whole blocks of 128 query rows: (name, kwargs for small_spec)
ROWS128_CASES = {
    "h128": dict(batch=5, heads=128, q_len=1, prefix_len=300, suffix_min=40, suffix_max=330,
                 seed=26),
    # 256 rows = two workgroups per request; the causal edge runs through the rows
    "h128_mtp": dict(batch=3, heads=128, q_len=2, prefix_len=70, suffix_min=1, suffix_max=200,
                     seed=41),
    # two query positions inside one workgroup's 128 rows, long enough for an odd number of steps
    "h64_qlen2": dict(batch=4, heads=64, q_len=2, prefix_len=130, suffix_min=60, suffix_max=450,
                      seed=42),
    "h128_block128": dict(batch=2, heads=128, q_len=1, prefix_len=33, suffix_min=0,
                          suffix_max=260, block_size=128, seed=43),
}


@pytest.mark.parametrize("chunk", [0, 64], ids=["auto_chunks", "chunk64"])
@pytest.mark.parametrize("mode", ["mixed", "absorb_only"])
@pytest.mark.parametrize("case", list(ROWS128_CASES))
def test_absorb_kernel_with_128_rows_per_workgroup(case, mode, chunk, gpu_device, tune):
    """The absorb kernel that gives a workgroup 128 query rows is chosen only for grids that cover
    the chip; debug flag 0x2000 takes it at any size.  Parity with the oracle, and agreement with
    the 64-row kernel (flag 0x1000) to the same tolerance."""
    if chunk:
        tune(T.TUNE_SUFFIX_CHUNK, chunk)
        tune(T.TUNE_ABSORB_PREFIX_CHUNK, chunk)
    wl = W.make_workload(W.small_spec(name=case, dtype="bf16", **ROWS128_CASES[case]))
    ref, ref_lse = O.mla_decode_definition(**wl.as_float64())
    print(f"128-row absorb kernel case={case} mode={mode} chunk={chunk}", flush=True)
    got, got_lse = Hh.run_library(wl, mode, gpu_device, flags=0x2000)
    Hh.assert_parity(got, got_lse, ref, ref_lse, "bf16", f"{case}/rows128/{mode}")
    other, other_lse = Hh.run_library(wl, mode, gpu_device, flags=0x1000)
    Hh.assert_parity(other, other_lse, ref, ref_lse, "bf16", f"{case}/rows64/{mode}")


ORDER_CASES = {
    # one per absorb kernel: <= 16, <= 32, 64 and 128 query rows per workgroup
    "h16": (dict(batch=9, heads=16, q_len=1, prefix_len=70, suffix_min=0, suffix_max=300,
                 seed=61), 0),
    "h32": (dict(batch=7, heads=32, q_len=1, prefix_len=40, suffix_min=1, suffix_max=200,
                 seed=62), 0),
    "h64_sq2": (dict(batch=6, heads=64, q_len=2, prefix_len=33, suffix_min=2, suffix_max=260,
                     seed=63), 0x1000),
    "h128": (dict(batch=5, heads=128, q_len=1, prefix_len=64, suffix_min=0, suffix_max=200,
                  seed=64), 0x2000),
}


@pytest.mark.parametrize("mode", ["mixed", "absorb_only"])
@pytest.mark.parametrize("case", list(ORDER_CASES))
def test_longest_suffix_first_order_changes_nothing(case, mode, gpu_device):
    """Grids with more workgroups than compute units start the requests with the longest suffix
    first (a small kernel ranks them); debug flag 0x4000 does so at any grid size, 0x8000 never.
    A request's result does not depend on when its workgroups run: parity with the oracle, and
    bit-identical to the run in batch order."""
    kw, kernel_flag = ORDER_CASES[case]
    wl = W.make_workload(W.small_spec(name="order_" + case, dtype="bf16", **kw))
    assert len(set(int(x) for x in wl.suffix_lens)) > 2     # ragged, with ties possible
    ref, ref_lse = O.mla_decode_definition(**wl.as_float64())
    print(f"longest-first order case={case} mode={mode}", flush=True)
    got, got_lse = Hh.run_library(wl, mode, gpu_device, flags=0x4000 | kernel_flag)
    Hh.assert_parity(got, got_lse, ref, ref_lse, "bf16", f"{case}/ordered/{mode}")
    plain, plain_lse = Hh.run_library(wl, mode, gpu_device, flags=0x8000 | kernel_flag)
    assert np.array_equal(got, plain, equal_nan=True)
    assert np.array_equal(got_lse, plain_lse, equal_nan=True)


@pytest.mark.parametrize("gain", [256.0, 16.0, 1.0 / 64.0])
def test_suffix_scores_far_from_the_first_step_128_rows(gain, gpu_device, tune):
    """test_suffix_scores_far_from_the_first_step for the 128-row absorb kernel, whose second
    walk takes exact maxima from a scores-only pass."""
    tune(T.TUNE_SUFFIX_CHUNK, 4096)
    spec = W.small_spec(name="suffix_growth_128", dtype="bf16", batch=4, heads=128, q_len=2,
                        prefix_len=40, suffix_min=200, suffix_max=700, seed=92)
    wl = W.make_workload(spec)
    wl.pool[:, :, 512:] *= gain
    for b in range(spec.batch):
        wl.pool[int(wl.block_table[b, 0]), :, 512:] /= gain     # the first 64 tokens stay
    ref, ref_lse = O.mla_decode_definition(**wl.as_float64())
    print(f"suffix score growth, 128-row kernel, gain={gain}", flush=True)
    for mode in ["mixed", "absorb_only"]:
        got, got_lse = Hh.run_library(wl, mode, gpu_device, flags=0x2000)
        Hh.assert_parity(got, got_lse, ref, ref_lse, "bf16", f"suffix_growth_128_{gain}/{mode}",
                         peaked=True)


@pytest.mark.parametrize("flags", [0, 0x1000, 0x2000], ids=["planned", "rows64", "rows128"])
@pytest.mark.parametrize("heads,batch,q_len,prefix,suffix,block",
                         [(16, 9, 1, 700, (0, 90), 64), (48, 5, 2, 129, (2, 300), 128),
                          (80, 3, 1, 64, (1, 65), 64), (32, 17, 3, 1000, (0, 0), 64),
                          (128, 2, 1, 63, (700, 700), 64)])
def test_absorb_prefix_over_the_rows_of_all_requests(heads, batch, q_len, prefix, suffix, block,
                                                     flags, gpu_device):
    """The latent prefix is walked for groups of 64 or 128 rows cut across requests: groups that
    end inside a request, a last group that is nearly empty, chunks that end inside a step, one
    launch for prefix and suffix or two (the flags), no suffix at all."""
    wl = W.make_workload(W.small_spec(dtype="bf16", batch=batch, heads=heads, q_len=q_len,
                                      prefix_len=prefix, suffix_min=suffix[0],
                                      suffix_max=suffix[1], block_size=block, seed=300 + batch))
    ref, ref_lse = O.mla_decode_definition(**wl.as_float64())
    print(f"absorb prefix rows={batch * q_len * heads} prefix={prefix} flags={flags:#x}", flush=True)
    got, got_lse = Hh.run_library(wl, "absorb_only", gpu_device, flags=flags)
    Hh.assert_parity(got, got_lse, ref, ref_lse, "bf16", f"absorb_prefix_{heads}x{batch}")


@pytest.mark.parametrize("heads,batch,q_len,prefix,suffix",
                         [(128, 4, 3, 1000, 2485), (96, 13, 3, 468, 499), (64, 14, 2, 2632, 632)])
def test_absorb_units_dealt_out_group_by_group(heads, batch, q_len, prefix, suffix, gpu_device):
    """Grids in which the suffix chunks beyond a multiple of 8 would give some XCDs a second round of
    workgroups: the row groups of those chunks are dealt out one by one.  Every row and every
    partial is written (the workspace starts out as NaN)."""
    wl = W.make_workload(W.small_spec(dtype="bf16", batch=batch, heads=heads, q_len=q_len,
                                      prefix_len=prefix, suffix_min=suffix // 2, suffix_max=suffix,
                                      seed=450 + batch))
    ref, ref_lse = O.mla_decode_absorb_all_heads(**wl.as_float64(),
                                                 requests=range(0, batch, max(1, batch // 4)))
    d = wl.to(gpu_device)
    dims = Hh.dims_of(wl)
    need = T.typhoon_mla_decode_workspace_bytes(dims, T.MODE_ABSORB_ONLY, batch, q_len, prefix,
                                                wl.max_suffix_len)
    ws = torch.full((need,), 255, dtype=torch.uint8, device=gpu_device)
    print(f"absorb grid {batch} x {q_len} x {heads}, {prefix} + {suffix}", flush=True)
    out, lse = T.typhoon_mla_decode(
        dims, "absorb_only", d.q, prefix, prefix_ckv=d.prefix_ckv, prefix_krope=d.prefix_krope,
        suffix_pool=d.pool, block_table=d.block_table, suffix_lens=d.suffix_lens,
        max_suffix_len=wl.max_suffix_len, w_uk=d.w_uk, w_uv=d.w_uv, workspace=ws)
    torch.cuda.synchronize(gpu_device)
    assert torch.isfinite(out).all() and torch.isfinite(lse).all()
    Hh.assert_parity(out.double().cpu().numpy(), lse.double().cpu().numpy(), ref, ref_lse, "bf16",
                     f"units_{heads}x{batch}")


@pytest.mark.parametrize("mode,dtype,heads,batch,kept_for,prefix,suffix",
                         [("mixed", "bf16", 16, 61, 64, 600, 500),
                          ("absorb_only", "bf16", 64, 14, 16, 600, 500),
                          ("absorb_only", "bf16", 16, 12, 16, 1500, 900),
                          ("auto", "bf16", 16, 12, 16, 1500, 900),
                          ("mixed", "bf16", 128, 3, 0, 300, 500),
                          ("absorb_only", "fp32", 16, 3, 0, 300, 300)])
def test_decode_within_a_workspace_kept_for_another_batch(mode, dtype, heads, batch, kept_for,
                                                          prefix, suffix, gpu_device):
    """The workspace named for a larger batch, where the smaller one prefers more (kept_for 0: just
    enough for one partial per part): same results, and nothing is written behind its end."""
    wl = W.make_workload(W.small_spec(dtype=dtype, batch=batch, heads=heads, q_len=1,
                                      prefix_len=prefix, suffix_min=suffix // 3, suffix_max=suffix,
                                      seed=77))
    dims, d = Hh.dims_of(wl), wl.to(gpu_device)
    n = wl.max_suffix_len
    wants = T.typhoon_mla_decode_workspace_bytes(dims, T.MODES[mode], batch, 1, prefix, n)
    if kept_for:
        kept = T.typhoon_mla_decode_workspace_bytes(dims, T.MODES[mode], kept_for, 1, prefix, n)
    else:
        esz = 2 if dtype == "bf16" else 4
        parts = 516 + 512 * esz + 4 if mode == "mixed" else 2 * (512 * esz + 4)
        kept = batch * heads * (576 * esz + parts) + 2048
    assert kept < wants
    pk, pv = T.typhoon_mla_expand_prefix(dims, d.prefix_ckv, d.prefix_krope, d.w_uk, d.w_uv)
    ws = torch.full((kept + 65536,), 255, dtype=torch.uint8, device=gpu_device)
    print(f"kept workspace {mode} {dtype} {batch} x {heads}: {kept} of {wants}", flush=True)
    out, lse = T.typhoon_mla_decode(
        dims, mode, d.q, prefix, prefix_k=pk, prefix_v=pv, prefix_ckv=d.prefix_ckv,
        prefix_krope=d.prefix_krope, suffix_pool=d.pool, block_table=d.block_table,
        suffix_lens=d.suffix_lens, max_suffix_len=n, w_uk=d.w_uk, w_uv=d.w_uv, workspace=ws[:kept])
    torch.cuda.synchronize(gpu_device)
    assert (ws[kept:] == 255).all()
    ref, ref_lse = O.mla_decode_definition(
        **wl.as_float64(), pairs=[(b, h) for b in range(0, batch, 5) for h in (0, heads - 1)])
    Hh.assert_parity(out.double().cpu().numpy(), lse.double().cpu().numpy(), ref, ref_lse, dtype,
                     f"kept_{mode}_{batch}")


@pytest.mark.parametrize("flags", [0, 1], ids=["mfma", "scalar"])
@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("ntok", [1, 31, 64, 100, 300])
def test_expand_prefix_matches_definition(dtype, ntok, flags, gpu_device):
    if dtype == "fp32" and flags == 1:
        pytest.skip("fp32 always runs the scalar kernels")
    wl = W.make_workload(W.small_spec(dtype=dtype, batch=1, heads=16, prefix_len=ntok,
                                      suffix_min=1, suffix_max=1, seed=40 + ntok))
    a = wl.as_float64()
    k_ref, v_ref = O.expand_prefix_definition(a["prefix_ckv"], a["prefix_krope"], a["w_uk"],
                                              a["w_uv"])
    d = wl.to(gpu_device)
    dims = Hh.dims_of(wl)
    print(f"expand dtype={dtype} ntok={ntok} flags={flags}", flush=True)
    old = T.typhoon_mla_set_debug_flags(flags)
    try:
        pk, pv = T.typhoon_mla_expand_prefix(dims, d.prefix_ckv, d.prefix_krope, d.w_uk, d.w_uv)
        torch.cuda.synchronize()
    finally:
        T.typhoon_mla_set_debug_flags(old)
    K, V = Hh.unpack_expanded(pk, pv, 16, ntok, dtype)
    rt = 2.0 ** -8 if dtype == "bf16" else 1e-5      # one bf16 rounding of an fp32 accumulation
    np.testing.assert_allclose(K, k_ref, rtol=rt, atol=1e-3 if dtype == "bf16" else 1e-6)
    np.testing.assert_allclose(V, v_ref, rtol=rt, atol=1e-3 if dtype == "bf16" else 1e-6)
    # the rope part is a verbatim copy
    np.testing.assert_array_equal(K[:, :, 128:], np.broadcast_to(a["prefix_krope"], (16, ntok, 64)))
    if dtype == "bf16" and ntok % 32:
        # padding tokens of the last 32-token block are zero
        kraw = pk.view(torch.bfloat16).double().cpu().numpy()
        hh, dd = np.meshgrid(np.arange(16), np.arange(192), indexing="ij")
        ntb32 = (ntok + 31) // 32 * 32
        for t in range(ntok, ntb32):
            assert np.all(kraw[Hh.k_offset(hh, ntb32, t, dd, dtype)] == 0)


@pytest.mark.parametrize("heads,ntok", [(128, 64), (128, 97), (128, 160), (128, 193), (128, 330),
                                        (16, 2700), (272, 70), (128, 700), (16, 5000)])
def test_expand_prefix_over_ranges_of_few_blocks(heads, ntok, gpu_device):
    """Workgroups of 1 to 6 and of 9 to 11 32-token blocks: odd and even walks, shorter than the ring
    of four slots and more than twice around it, a ragged last block at the end of either, more
    heads than compute units.  Bounds as above: one bf16 rounding of an fp32
    accumulation over 512 products."""
    wl = W.make_workload(W.small_spec(dtype="bf16", batch=1, heads=heads, prefix_len=ntok,
                                      suffix_min=1, suffix_max=1, seed=140 + ntok))
    a = wl.as_float64()
    k_ref, v_ref = O.expand_prefix_definition(a["prefix_ckv"], a["prefix_krope"], a["w_uk"],
                                              a["w_uv"])
    d = wl.to(gpu_device)
    print(f"expand heads={heads} ntok={ntok}", flush=True)
    pk, pv = T.typhoon_mla_expand_prefix(Hh.dims_of(wl), d.prefix_ckv, d.prefix_krope, d.w_uk,
                                         d.w_uv)
    K, V = Hh.unpack_expanded(pk, pv, heads, ntok, "bf16")
    np.testing.assert_allclose(K, k_ref, rtol=2.0 ** -8, atol=1e-3)
    np.testing.assert_allclose(V, v_ref, rtol=2.0 ** -8, atol=1e-3)
    if ntok % 32:   # the last block of every head: zeros behind the last token
        ntb = (ntok + 31) // 32
        kb = pk.view(torch.bfloat16).view(heads, ntb, 12, 2, 32, 8)[:, -1]
        vb = pv.view(torch.bfloat16).view(heads, ntb, 2, 4, 2, 32, 8)[:, -1]
        assert kb[:, :, :, ntok % 32:].abs().max() == 0
        tok = torch.arange(32).view(2, 2, 2, 4)    # [16-token half, 8-token half, lane half, 4]
        tok = tok.permute(0, 2, 1, 3).reshape(2, 1, 2, 1, 8).to(gpu_device)
        assert torch.where(tok >= ntok % 32, vb.float(), torch.zeros_like(vb, dtype=torch.float32)
                           ).abs().max() == 0


@pytest.mark.parametrize("heads,ntok", [(16, 32), (16, 255), (16, 600), (16, 1003), (16, 1790), (32, 620),
                                        (48, 200), (64, 300), (64, 437)])
def test_expand_prefix_with_k_and_v_apart(heads, ntok, gpu_device):
    """Workgroups that expand a head's K or its V only: 1 to 7 blocks, the same bounds."""
    test_expand_prefix_over_ranges_of_few_blocks(heads, ntok, gpu_device)


@pytest.mark.parametrize("out_dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("n,rows,width", [(1, 5, 128), (3, 130, 128), (7, 33, 512), (2, 1, 4)])
def test_combine_lse_matches_definition(n, rows, width, out_dtype, gpu_device):
    g = torch.Generator().manual_seed(n * 1000 + rows)
    po = torch.randn((n, rows, width), generator=g)
    pl = torch.randn((n, rows), generator=g) * 4
    # sprinkle empty partials (LSE = -inf with NaN payload) and one fully empty row
    pl[0, ::3] = float("-inf")
    po[0, ::3] = float("nan")
    if rows > 1:
        pl[:, 1] = float("-inf")
    ref_o, ref_l = O.combine_lse(po.double().numpy(), pl.double().numpy())
    print(f"combine n={n} rows={rows} width={width} {out_dtype}", flush=True)
    out, lse = T.typhoon_mla_combine_lse(po.to(gpu_device), pl.to(gpu_device), out_dtype)
    torch.cuda.synchronize()
    tol = 1e-5 if out_dtype == torch.float32 else 2.0 ** -8
    np.testing.assert_allclose(out.double().cpu().numpy(), ref_o, rtol=tol, atol=1e-6)
    got_l = lse.double().cpu().numpy()
    assert np.array_equal(np.isneginf(got_l), np.isneginf(ref_l))
    fin = np.isfinite(ref_l)
    np.testing.assert_allclose(got_l[fin], ref_l[fin], atol=1e-5, rtol=1e-6)


@pytest.mark.parametrize("mode", ["mixed", "absorb_only"])
def test_large_batch_projection_kernels(mode, gpu_device):
    """More than 1024 queries per head at 64 heads: the query absorption stages a weight slice once
    for four blocks of 128 queries, with a ragged last group (1100 = 8 x 128 + 76 = 34 x 32 + 12
    queries), and the projection takes seven runs of five blocks of 32 a head, in two rounds of
    workgroups.  Every row against the tensor-form absorb checker, a sample against the definition."""
    spec = W.small_spec(name="large_batch_h64", dtype="bf16", batch=1100, heads=64, q_len=1,
                        prefix_len=64, suffix_min=0, suffix_max=24, seed=55)
    wl = W.make_workload(spec)
    a = wl.as_float64()
    ref2, ref2_lse = Hh.oracle_absorb_all_heads_parallel(O, a)
    pairs = [(b, h) for b in (0, 1, 511, 1023, 1024, 1099) for h in (0, 31, 63)]
    ref, ref_lse = O.mla_decode_definition(**a, pairs=pairs)
    print(f"large batch projections mode={mode}", flush=True)
    got, got_lse = Hh.run_library(wl, mode, gpu_device)
    Hh.assert_parity(got, got_lse, ref2, ref2_lse, "bf16", f"large_batch/{mode}/absorb-form")
    Hh.assert_parity(got, got_lse, ref, ref_lse, "bf16", f"large_batch/{mode}/definition")


def test_projection_with_two_naive_partials(gpu_device):
    """200 requests x 128 heads: the prefix pass splits its tokens in two (two naive partials per
    row), and the projection takes runs of 4 and 3 blocks of 32 queries through its ring, the last
    block with 8 valid rows.  Some requests have no suffix at all (their
    latent partial is never written and must count as zeros)."""
    spec = W.small_spec(name="two_naive_partials_h128", dtype="bf16", batch=200, heads=128, q_len=1,
                        prefix_len=160, suffix_min=0, suffix_max=20, seed=77)
    wl = W.make_workload(spec)
    a = wl.as_float64()
    ref2, ref2_lse = Hh.oracle_absorb_all_heads_parallel(O, a)
    pairs = [(b, h) for b in (0, 95, 96, 191, 192, 199) for h in (0, 64, 127)]
    ref, ref_lse = O.mla_decode_definition(**a, pairs=pairs)
    print("projection, two naive partials", flush=True)
    got, got_lse = Hh.run_library(wl, "mixed", gpu_device)
    Hh.assert_parity(got, got_lse, ref2, ref2_lse, "bf16", "two_naive/absorb-form")
    Hh.assert_parity(got, got_lse, ref, ref_lse, "bf16", "two_naive/definition")


@pytest.mark.parametrize("mode", MODES)
def test_bitwise_repeatable(mode, gpu_device):
    wl, _ = _workload_and_ref("ragged_h16", "bf16")
    a = Hh.run_library(wl, mode, gpu_device)
    b = Hh.run_library(wl, mode, gpu_device)
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])


@pytest.mark.parametrize("mode", MODES)
def test_cfg1_tiny_fp32_full(mode, gpu_device):
    wl = W.make_workload(W.CONFIGS["cfg1_tiny_fp32"])
    ref, ref_lse = O.mla_decode_definition(**wl.as_float64())
    print(f"cfg1 mode={mode}", flush=True)
    got, got_lse = Hh.run_library(wl, mode, gpu_device)
    Hh.assert_parity(got, got_lse, ref, ref_lse, "fp32", f"cfg1/{mode}")


def test_modes_agree_with_each_other(gpu_device):
    wl, _ = _workload_and_ref("mtp_h32", "bf16")
    outs = {m: Hh.run_library(wl, m, gpu_device) for m in MODES}
    for m in MODES[1:]:
        np.testing.assert_allclose(outs[m][0], outs["mixed"][0], atol=1e-2, rtol=2e-2)
        fin = np.isfinite(outs["mixed"][1])
        np.testing.assert_allclose(outs[m][1][fin], outs["mixed"][1][fin], atol=2e-3)


AUTO_CASES = {
    # below the break-even batch of 128 heads and a 2048-token prefix (62): absorb_only runs
    "below_break_even": dict(batch=2, heads=128, q_len=1, prefix_len=2048, suffix_min=10,
                             suffix_max=120, seed=51),
    # above that of 32 heads (194; the batches here were 40 and 20 while the table's was 32): mixed runs
    "above_break_even": dict(batch=200, heads=32, q_len=1, prefix_len=2048, suffix_min=0,
                             suffix_max=60, seed=52),
    # two query positions per request halve it (97)
    "above_with_two_queries": dict(batch=100, heads=32, q_len=2, prefix_len=2048, suffix_min=2,
                                   suffix_max=60, seed=53),
}


@pytest.mark.parametrize("case", list(AUTO_CASES))
def test_auto_mode_matches_oracle(case, gpu_device):
    wl = W.make_workload(W.small_spec(name=case, dtype="bf16", **AUTO_CASES[case]))
    spec = wl.spec
    thr = T.typhoon_mla_auto_batch_threshold(Hh.dims_of(wl), spec.q_len, spec.prefix_len)
    assert (spec.batch < thr) == (case == "below_break_even")
    ref, ref_lse = O.mla_decode_definition(**wl.as_float64())
    print(f"auto mode case={case} threshold={thr:.2f}", flush=True)
    got, got_lse = Hh.run_library(wl, "auto", gpu_device)
    Hh.assert_parity(got, got_lse, ref, ref_lse, "bf16", f"{case}/auto")
    # auto is exactly the mode it resolves to
    same, same_lse = Hh.run_library(wl, "absorb_only" if spec.batch < thr else "mixed", gpu_device)
    assert np.array_equal(got, same) and np.array_equal(got_lse, same_lse)


@pytest.mark.parametrize("case,flags", [("h128_many_tiles", 0), ("ragged_h16", 0),
                                        ("h128_many_tiles", 0x2000)],
                         ids=["h128", "h16", "h128_rows128"])
def test_decode_replays_from_a_hip_graph(case, flags, gpu_device):
    """The library only enqueues kernels on the caller's stream (no allocation, no host
    synchronisation, no memset nodes), so a decode step can be captured into a HIP graph.  Every
    replay, with eager work and synchronisations in between, must reproduce the eager result bit
    for bit, also after the inputs have changed in place."""
    wl, (ref, ref_lse) = _workload_and_ref(case, "bf16")
    d = wl.to(gpu_device)
    dims = Hh.dims_of(wl)
    L_s = wl.spec.prefix_len
    pk, pv = T.typhoon_mla_expand_prefix(dims, d.prefix_ckv, d.prefix_krope, d.w_uk, d.w_uv)
    B, S, H = wl.spec.batch, wl.spec.q_len, wl.spec.heads
    out = torch.empty((B, S, H, 128), dtype=torch.bfloat16, device=gpu_device)
    lse = torch.empty((B, S, H), dtype=torch.float32, device=gpu_device)
    nbytes = T.typhoon_mla_decode_workspace_bytes(dims, T.MODE_MIXED, B, S, L_s, wl.max_suffix_len)
    ws = torch.empty(max(nbytes, 256), dtype=torch.uint8, device=gpu_device)
    q = d.q.clone()

    def step():
        T.typhoon_mla_decode(dims, "mixed", q, L_s, prefix_k=pk, prefix_v=pv,
                             suffix_pool=d.pool, block_table=d.block_table,
                             suffix_lens=d.suffix_lens, max_suffix_len=wl.max_suffix_len,
                             w_uk=d.w_uk, w_uv=d.w_uv, out=out, lse_out=lse, workspace=ws)

    print(f"graph capture case={case} flags={flags:#x}", flush=True)
    old_flags = T.typhoon_mla_set_debug_flags(flags)   # 0x2000: the 128-row absorb kernel
    try:
        step()                                   # eager: also performs the one-time kernel set-up
        torch.cuda.synchronize(gpu_device)
        eager = (out.clone(), lse.clone())
        Hh.assert_parity(out.double().cpu().numpy(), lse.double().cpu().numpy(), ref, ref_lse, "bf16",
                         f"{case}/eager")
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            step()
        for rep in range(3):
            out.fill_(float("nan"))              # eager work between replays
            lse.fill_(float("nan"))
            torch.cuda.synchronize(gpu_device)
            graph.replay()
            torch.cuda.synchronize(gpu_device)
            assert torch.equal(out, eager[0]) and torch.equal(lse, eager[1]), f"replay {rep} differs"
        # new queries written in place are picked up by the next replay
        q.copy_(torch.flip(d.q, dims=[0]))
        graph.replay()
        torch.cuda.synchronize(gpu_device)
        flipped = (out.clone(), lse.clone())
        step()
        torch.cuda.synchronize(gpu_device)
        assert torch.equal(out, flipped[0]) and torch.equal(lse, flipped[1])
    finally:
        T.typhoon_mla_set_debug_flags(old_flags)
