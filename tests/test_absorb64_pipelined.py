"""The software-pipelined absorb kernel with 64 query rows per workgroup: chunks of one to six tiles of 32 tokens with every
remainder that its ring of four treats differently, partial row groups, the causal edge, and the wait states
around its assembly MFMAs."""
import os
import re
import subprocess

import numpy as np
import pytest
import torch

from oracle import mla_oracle as O
from paper_2509_21081_amd import binding as T
from paper_2509_21081_amd import build as B
from paper_2509_21081_amd import workloads as W
from tests import helpers as Hh
from tests import test_isa_hazards as hz

# (tokens, heads, q_len): one tile and parts of it, the first with a prefetched tile, the last partial; 48 and
# 96 rows leave row blocks that are partly or wholly no request's
SHAPES = [(1, 48, 1), (31, 48, 1), (32, 64, 1), (33, 48, 2), (64, 64, 2), (65, 48, 1), (96, 64, 1), (97, 48, 3),
          (127, 64, 1), (128, 48, 4), (129, 80, 1), (160, 64, 1), (161, 96, 1), (192, 64, 4)]


@pytest.mark.gpu
@pytest.mark.parametrize("tokens,heads,q_len", SHAPES)
def test_tiles_and_their_remainders(tokens, heads, q_len, gpu_device, tune):
    # one chunk of 192 tokens a request, of which it has `tokens` (chunks of up to 128 are another kernel's); the
    # prefix in one such chunk and one of 33 tokens
    tune(T.TUNE_SUFFIX_CHUNK, 192)
    tune(T.TUNE_ABSORB_PREFIX_CHUNK, 192)
    wl = W.make_workload(W.small_spec(name="tiles", dtype="bf16", batch=3, heads=heads, q_len=q_len, prefix_len=225,
                                      suffix_min=192, suffix_max=192, seed=tokens))
    wl.suffix_lens.fill_(max(tokens, q_len))
    ref, ref_lse = O.mla_decode_definition(**wl.as_float64())
    for mode in ["mixed", "absorb_only"]:
        for flags in [0x1000, 0x1800]:   # the 64-row kernel; its exact walk
            print(f"64-row pipelined kernel {tokens} x {heads} x {q_len} {mode} {flags:#x}", flush=True)
            got, got_lse = Hh.run_library(wl, mode, gpu_device, flags=flags)
            Hh.assert_parity(got, got_lse, ref, ref_lse, "bf16", f"tiles/{tokens}/{heads}/{q_len}/{mode}/{flags:#x}")


@pytest.mark.gpu
@pytest.mark.parametrize("batch,prefix", [(255, 64), (256, 64), (256, 0)])
def test_both_sides_of_the_line_to_the_kernel_of_64_token_steps(batch, prefix, gpu_device, tune):
    tune(T.TUNE_SUFFIX_CHUNK, 192)
    wl = W.make_workload(W.small_spec(name="line", dtype="bf16", batch=batch, heads=64, q_len=1, prefix_len=prefix,
                                      suffix_min=1, suffix_max=110, seed=batch + prefix))
    # (chunks of 192 tokens: up to 128 the other kernel takes any grid)
    wl.block_table = torch.nn.functional.pad(wl.block_table, (0, 1))
    wl.max_suffix_len = 192
    ref, ref_lse = O.mla_decode_definition(**wl.as_float64())
    print(f"64-row kernels batch={batch} prefix={prefix}", flush=True)
    got, got_lse = Hh.run_library(wl, "mixed", gpu_device)
    Hh.assert_parity(got, got_lse, ref, ref_lse, "bf16", f"line/{batch}/{prefix}")


@pytest.mark.gpu
@pytest.mark.parametrize("token", [5, 40, 100, 150, 191, 200])
def test_a_nan_takes_its_whole_chunk(token, gpu_device, tune):
    """Chunks of 192 and 108 tokens: a key that scores NaN takes the whole chunk with it, in whichever tile it is, and no
    other chunk or request."""
    tune(T.TUNE_SUFFIX_CHUNK, 192)
    wl = W.make_workload(W.small_spec(name="nan_tiles", dtype="bf16", batch=3, heads=64, q_len=1, prefix_len=64,
                                      suffix_min=300, suffix_max=300, seed=971))
    clean, clean_lse = Hh.run_library(wl, "mixed", gpu_device)
    assert np.isfinite(clean).all() and np.isfinite(clean_lse).all()
    a = wl.as_float64()
    table = a["block_table"][1]
    wl.pool[table[token // 64], token % 64, 570] = float("nan")
    if token < 192:     # the second chunk is left, its 108 tokens in front
        whole = a["pool"].copy()
        for i in range(108):
            a["pool"][table[i // 64], i % 64] = whole[table[(192 + i) // 64], (192 + i) % 64]
    a["suffix_lens"] = np.array([300, 108 if token < 192 else 192, 300])
    ref, ref_lse = O.mla_decode_definition(**a, pairs=[(1, h) for h in range(0, 64, 5)])
    print(f"NaN at suffix token {token}", flush=True)
    got, got_lse = Hh.run_library(wl, "mixed", gpu_device)
    Hh.assert_parity(got, got_lse, ref, ref_lse, "bf16", f"nan_tiles/{token}")
    assert np.array_equal(got[[0, 2]], clean[[0, 2]]) and np.array_equal(got_lse[[0, 2]], clean_lse[[0, 2]])


@pytest.mark.gpu
@pytest.mark.parametrize("suffix", [4097, 4300])
def test_a_chunk_of_more_blocks_than_lanes(suffix, gpu_device, tune):
    """One chunk of 65 and of 68 cache blocks: a lane holds each of the first 64 entries of the block table, the others are
    loaded one by one."""
    tune(T.TUNE_SUFFIX_CHUNK, 4352)
    wl = W.make_workload(W.small_spec(name="blocks", dtype="bf16", batch=2, heads=64, q_len=1, prefix_len=0,
                                      suffix_min=suffix, suffix_max=suffix, seed=suffix))
    ref, ref_lse = O.mla_decode_definition(**wl.as_float64(), pairs=[(b, h) for b in (0, 1) for h in (0, 21, 63)])
    for flags in [0, 0x800]:
        print(f"one chunk of {suffix} tokens, flags {flags:#x}", flush=True)
        got, got_lse = Hh.run_library(wl, "mixed", gpu_device, flags=flags)
        Hh.assert_parity(got, got_lse, ref, ref_lse, "bf16", f"blocks/{suffix}/{flags:#x}")


def decode_absorb(heads, batch, prefix, suffix, device):
    """absorb_only step of the first `batch` of the same 256 requests"""
    wl = W.make_workload(W.small_spec(name="dispatch", dtype="bf16", batch=256, heads=heads, q_len=1, prefix_len=prefix,
                                      suffix_min=suffix, suffix_max=suffix, seed=heads))
    wl.q, wl.block_table, wl.suffix_lens = wl.q[:batch], wl.block_table[:batch], wl.suffix_lens[:batch]
    print(f"dispatch {heads} x {batch} over {prefix} + {suffix}", flush=True)
    return Hh.run_library(wl, "absorb_only", device)


@pytest.mark.gpu
@pytest.mark.parametrize("heads", [16, 32])
def test_joint_launches_of_few_rows_stay_with_the_pipelined_kernel(heads, gpu_device, tune):
    """Prefix and suffixes in one launch, on both sides of 256 workgroups: the two 64-row kernels round differently (16x16
    and 32x32 products, references of 32 and 64 tokens), so equal bits mean the same kernel.  (The other
    one made the absorb form 9 % slower than mixed mode where auto mode takes it, at 128 x 16 heads over 4096 + 512 tokens.)"""
    tune(T.TUNE_SUFFIX_CHUNK, 192)
    tune(T.TUNE_ABSORB_PREFIX_CHUNK, 192)
    # 192 + 192 tokens in a chunk each: 16 heads 51 + 204 = 255 and 52 + 208, 32 heads 84 + 168 and 86 + 172
    few, many = {16: (204, 208), 32: (168, 172)}[heads]
    small, small_lse = decode_absorb(heads, few, 192, 192, gpu_device)
    large, large_lse = decode_absorb(heads, many, 192, 192, gpu_device)
    assert np.array_equal(small, large[:few]) and np.array_equal(small_lse, large_lse[:few])


def decode_mixed(batch, prefix, suffix, device):
    """mixed step of the first `batch` of the same 257 requests x 64 heads"""
    wl = W.make_workload(W.small_spec(name="lines", dtype="bf16", batch=257, heads=64, q_len=1, prefix_len=prefix,
                                      suffix_min=suffix, suffix_max=suffix, seed=7))
    wl.q, wl.block_table, wl.suffix_lens = wl.q[:batch], wl.block_table[:batch], wl.suffix_lens[:batch]
    wl.block_table = torch.nn.functional.pad(wl.block_table, (0, 4 - wl.block_table.shape[1]))
    wl.max_suffix_len = 256
    print(f"line {batch} x 64 over {prefix} + {suffix}", flush=True)
    return Hh.run_library(wl, "mixed", device)


@pytest.mark.gpu
def test_which_kernel_a_launch_takes(gpu_device, tune):
    """By equal and different bits, as above: 64 rows a request beside a prefix pass go back to the kernel of 64-token steps
    from 256 workgroups on, without a prefix they do not, and chunks of up to 128 tokens always do."""
    def same(x, y):
        n = min(len(x[0]), len(y[0]))
        return np.array_equal(x[0][:n], y[0][:n]) and np.array_equal(x[1][:n], y[1][:n])
    tune(T.TUNE_SUFFIX_CHUNK, 256)
    a, b, c = (decode_mixed(n, 64, 160, gpu_device) for n in (254, 255, 256))
    assert same(a, b) and not same(b, c)
    assert same(decode_mixed(255, 0, 160, gpu_device), decode_mixed(256, 0, 160, gpu_device))
    # 100 tokens, one chunk of 256, 192 and 128
    runs = []
    for chunk in (256, 192, 128):
        tune(T.TUNE_SUFFIX_CHUNK, chunk)
        runs.append(decode_mixed(40, 0, 100, gpu_device))
    assert same(runs[0], runs[1]) and not same(runs[0], runs[2])


@pytest.mark.skipif(not os.path.exists(B.HIPCC), reason="hipcc not available")
def test_wait_states_of_the_assembly_mfmas(tmp_path):
    out = tmp_path / "k.s"
    subprocess.run([B.HIPCC, *B.FLAGS, "-S", "--cuda-device-only", "-o", str(out),
                    os.path.join(B.CSRC, "tmla_absorb64_pipelined_mfma.hip")], check=True, capture_output=True)
    text = out.read_text()
    kernel = "absorb64_pipelined_kernel"
    starts = [m.start() for m in re.finditer(r"\n_ZN4tmla%d%sI[^:\s]*:" % (len(kernel), kernel), text)]
    assert len(starts) == 2
    for start in starts:
        instrs, labels = [], {}
        for raw in text[start:text.index("\n.Lfunc_end", start)].split("\n"):
            t = raw.split(";")[0].strip()
            if t.endswith(":"):
                labels[t[:-1]] = len(instrs)
            elif t and not t.startswith("."):
                instrs.append(t)
        for where, seq in hz._sequences(instrs, labels):
            hz._check_valu_to_mfma(seq, where)
            hz._check_mfma_result(seq, where)
        assert sum(i.startswith("v_mfma") for i in instrs) > 100
