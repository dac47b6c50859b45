"""GPU parity: the HIP path, called through the C ABI, against the CPU oracle on the same
seeded inputs.  Integers (positions, slots, masks) bit-exact; outputs within 1e-4 max-abs
(fp32) or 2e-2 x RMS (bf16)."""
import numpy as np
import pytest
import torch

from oracle import hpd_oracle as O
from paper_2604_26209_amd import workloads as W

import hpd_harness as H

pytestmark = pytest.mark.gpu


def _say(msg):
    print(msg, flush=True)


def _us_in_turn(calls):
    """us per call of each of the calls, timed in turn: the least of five times ten."""
    us = [1e9] * len(calls)
    for _ in range(5):
        for i, call in enumerate(calls):
            call()
            start, end = torch.cuda.Event(True), torch.cuda.Event(True)
            start.record()
            for _ in range(10):
                call()
            end.record()
            torch.cuda.synchronize()
            us[i] = min(us[i], start.elapsed_time(end) * 100)
    return us


def test_cfg1_fp32_all_steps_two_call_and_fused():
    wl = W.config(1)
    _say("cfg1 two-call")
    hip = H.run_hip(wl)
    err = H.check_all(wl, hip, label="cfg1")
    _say(f"cfg1 max-abs {err:.2e}")
    _say("cfg1 fused")
    hip2 = H.run_hip(wl, inputs=hip["inputs"], fused=True)
    for a, b in zip(hip["out"], hip2["out"]):
        assert torch.equal(a, b)


@pytest.mark.parametrize("seed", [1, 2, 3])
def test_random_ragged_fp32(seed):
    _say(f"random fp32 seed {seed}")
    wl = W.random_workload(seed, dtype="f32", hq=4, hkv=2, d=64, t=6, p=3)
    hip = H.run_hip(wl)
    H.check_all(wl, hip, label=f"rand_f32_{seed}")


def test_fp32_other_head_dims_and_empty_header():
    for d, hq, hkv in [(32, 2, 1), (128, 4, 4), (96, 3, 1)]:
        _say(f"fp32 D={d}")
        wl = W.random_workload(40 + d, dtype="f32", hq=hq, hkv=hkv, d=d, t=3, p=2, h_range=(0, 0),
                               l_range=(1, 40))
        H.check_all(wl, H.run_hip(wl), label=f"f32_D{d}")


@pytest.mark.parametrize("mode", [1, 2, 3, 4])
@pytest.mark.parametrize("seed", [11, 12])
def test_random_ragged_bf16_both_kernels(seed, mode):
    """mode 1 = generic wave-reduction kernel, 2 = LDS-streaming MFMA kernel (the default for
    this shape), 3 / 4 = the same with the wide / narrow workgroup shape forced."""
    _say(f"random bf16 seed {seed} mode {mode}")
    wl = W.random_workload(seed, dtype="bf16", hq=8, hkv=2, d=128, base=500000.0, t=5, p=3,
                           h_range=(0, 70), l_range=(1, 150), n_range=(1, 12))
    hip = H.run_hip(wl, kernel_mode=mode)
    rel = H.check_all(wl, hip, label=f"rand_bf16_{seed}_m{mode}")
    _say(f"  worst err/rms {rel:.2e}")


@pytest.mark.parametrize("mode", [3, 4])
@pytest.mark.parametrize("g", [1, 2, 4, 8])
def test_stream_kernel_fused_step_equals_two_calls(g, mode):
    """hpd_decode_step (one launch, append inside the attention kernel) against
    hpd_kv_append + hpd_decode_attention: same tail pools, same outputs, bit for bit."""
    _say(f"stream fused vs two-call G={g} mode {mode}")
    wl = W.random_workload(60 + g, dtype="bf16", hq=8, hkv=8 // g, d=128, base=500000.0, t=6, p=3,
                           h_range=(0, 90), l_range=(1, 300), n_range=(1, 14))
    a = H.run_hip(wl, kernel_mode=mode, fused=False, poison_pools="zero")
    b = H.run_hip(wl, inputs=a["inputs"], kernel_mode=mode, fused=True, poison_pools="zero")
    for x, y in zip(a["out"], b["out"]):
        assert torch.equal(x, y)
    for x, y in zip(a["pools"][2:], b["pools"][2:]):
        assert torch.equal(x, y)
    rel = H.check_all(wl, b, label=f"stream_fused_g{g}")
    _say(f"  worst err/rms {rel:.2e}")


@pytest.mark.parametrize("seed", range(100, 108))
def test_random_layout_sweep_stream_kernel(seed):
    """Random small batches through the step call: group size, head count, number of steps
    (up to four chunks of tail positions), ragged lengths, document and branch counts all
    drawn from the seed; all workgroup shapes."""
    rng = np.random.default_rng(seed)
    g = int(rng.choice([1, 2, 4, 8]))
    hkv = int(rng.choice([1, 2, 4]))
    t = int(rng.integers(1, 27))
    wl = W.random_workload(seed, dtype="bf16", hq=hkv * g, hkv=hkv, d=128, base=500000.0, t=t,
                           p=int(rng.integers(1, 4)), j_range=(1, 3), n_range=(1, int(rng.integers(2, 40))),
                           h_range=(0, int(rng.integers(1, 100))), l_range=(1, int(rng.integers(2, 400))))
    for mode in (3, 4):
        _say(f"sweep seed {seed}: G={g} Hkv={hkv} T={t} branches={wl.n_branches} mode {mode}")
        hip = H.run_hip(wl, kernel_mode=mode, fused=True)
        H.check_all(wl, hip, label=f"sweep_{seed}_m{mode}")


@pytest.mark.parametrize("mode", [3, 4])
@pytest.mark.parametrize("case", ["tiny_prefix", "many_branches", "no_header_one_key"])
def test_tail_tile_formats_of_the_newest_chunk(case, mode):
    """The newest chunk of tail positions is cut into tiles of 1 x 32, 2 x 16, 4 x 8 or 8 x 4
    (positions x branches) depending on how many positions it holds: every step 0..11 goes through
    each format at least once, with full chunks behind it from step 8 on.  Cases: prefixes so short
    that a tile of the newest chunk is among the first requests (its row table is then written
    before the loaders start); documents with more branches than one tile or one row block holds
    (tiles that span row blocks, ragged last tile); no header and a one-token document.  Every
    group size; fused = two-call bit for bit; against the oracle."""
    kw = dict(tiny_prefix=dict(p=3, j_range=(1, 3), n_range=(1, 40), h_range=(0, 20), l_range=(1, 40)),
              many_branches=dict(p=2, j_range=(1, 2), n_range=(30, 70), h_range=(0, 70), l_range=(1, 300)),
              no_header_one_key=dict(p=2, j_range=(1, 3), n_range=(1, 35), h_range=(0, 0), l_range=(1, 1)))[case]
    for g in (1, 2, 4, 8):
        _say(f"tile formats: {case} G={g} mode {mode}")
        wl = W.random_workload(300 + g, dtype="bf16", hq=8, hkv=8 // g, d=128, base=500000.0, t=12, **kw)
        a = H.run_hip(wl, kernel_mode=mode, fused=True)
        rel = H.check_all(wl, a, label=f"fmt_{case}_g{g}_m{mode}")
        b = H.run_hip(wl, inputs=a["inputs"], kernel_mode=mode, fused=False)
        for x, y in zip(a["out"], b["out"]):
            assert torch.equal(x, y)
        _say(f"  worst err/rms {rel:.2e}")


@pytest.mark.parametrize("mode", [1, 3, 4])
@pytest.mark.parametrize("case", ["peaked_x4", "argmax_x16", "flat_div16", "common_offset", "rising"])
def test_score_ranges_of_the_online_softmax(case, mode):
    """Inputs other than N(0,1): scores 4 and 16 times as wide (rows that one or two keys
    dominate, up to an argmax), 16 times as narrow (a flat average), with a large common
    component in queries and keys (every score near +16 in log2 units: the reference point of
    the exponentials must follow), and with keys that grow along the document and the steps (the
    maximum of a row keeps rising, block after block: the accumulators are rescaled again and
    again).  Same tolerance as everywhere; generic kernel (mode 1) and all workgroup shapes."""
    wl = W.random_workload(400, dtype="bf16", hq=8, hkv=2, d=128, base=500000.0, t=11, p=2,
                           j_range=(1, 3), n_range=(1, 20), h_range=(0, 70), l_range=(40, 400))
    from paper_2604_26209_amd import binding as B
    lay = B.layout_from_workload(wl)
    inp = H.Inputs(wl, lay.n_live(), "cuda", lay.counts()[B.HPD_C_N_PREFIX_TOKENS])
    bf = lambda x: x.float().to(torch.bfloat16)
    if case in ("peaked_x4", "argmax_x16", "flat_div16"):
        f = dict(peaked_x4=4.0, argmax_x16=16.0, flat_div16=1.0 / 16)[case]
        inp.q = [bf(x.float() * f) for x in inp.q]
    elif case == "common_offset":
        inp.q = [bf(x.float() + 1.0) for x in inp.q]
        inp.k_raw = bf(inp.k_raw.float() + 1.0)
        inp.k_new = [bf(x.float() + 1.0) for x in inp.k_new]
    else:
        # a component along which all queries point and the keys grow with their index
        n = inp.k_raw.shape[0]
        ramp = torch.arange(n, device="cuda", dtype=torch.float32)[:, None, None] * (4.0 / max(n, 1))
        inp.k_raw = bf(inp.k_raw.float() + ramp)
        inp.k_new = [bf(x.float() + 4.0 + 0.3 * t) for t, x in enumerate(inp.k_new)]
        inp.q = [bf(x.float() * 0.5 + 1.0) for x in inp.q]
    _say(f"score ranges: {case} mode {mode}")
    a = H.run_hip(wl, inputs=inp, kernel_mode=mode, fused=mode != 1)
    rel = H.check_all(wl, a, label=f"{case}_m{mode}")
    _say(f"  worst err/rms {rel:.2e}")


def test_values_beyond_the_half_range_saturate():
    """The pools hold their bf16 values in half format, which ends at 65504: keys and values of
    larger magnitude (bf16 can carry them) are stored as +-65504.  Nothing overflows - every output
    stays finite, also in the rows that attend to such elements -, and the prompts without such
    elements are unaffected (same tolerance against the oracle as ever)."""
    wl = W.random_workload(410, dtype="bf16", hq=8, hkv=2, d=128, base=500000.0, t=6, p=3,
                           j_range=(1, 3), n_range=(2, 12), h_range=(10, 70), l_range=(40, 200))
    from paper_2604_26209_amd import binding as B
    lay = B.layout_from_workload(wl)
    inp = H.Inputs(wl, lay.n_live(), "cuda", lay.counts()[B.HPD_C_N_PREFIX_TOKENS])
    # prompt 0 only: a few huge elements in its header, its first document and its new rows
    h0 = int(wl.header_len[0])
    big = torch.tensor(1.0e5, dtype=torch.bfloat16, device="cuda")
    inp.k_raw[1, 0, 5] = big
    inp.k_raw[h0 + 3, 1, 70] = -big
    inp.v_raw[2, 0, 9] = big
    inp.v_raw[h0 + 4, 1, 100] = -big
    inp.k_new[0][0, 0, 17] = big
    inp.v_new[1][0, 1, 3] = big
    for mode in (3, 4):
        _say(f"saturation mode {mode}")
        a = H.run_hip(wl, inputs=inp, kernel_mode=mode, fused=True)
        for o in a["out"]:
            assert bool(torch.isfinite(o.float()).all())
        H.check_all(wl, a, prompts=[1, 2], label=f"saturate_m{mode}")


@pytest.mark.parametrize("g", [3, 5, 6, 7])
def test_stream_kernel_group_sizes_that_are_not_powers_of_two(g):
    """Group sizes such as 40 query heads over 8 kv heads (5) run on the streaming kernel with
    the rows of a branch padded to the next power of two; padding rows are neither loaded nor
    stored.  Decode (both masks, fused = two-call) and prefill, all workgroup shapes."""
    rng = np.random.default_rng(190 + g)
    hkv = int(rng.choice([1, 2]))
    wl = W.random_workload(190 + g, dtype="bf16", hq=hkv * g, hkv=hkv, d=128, base=500000.0,
                           t=int(rng.integers(2, 20)), p=3, j_range=(1, 3), n_range=(1, 30),
                           h_range=(0, 100), l_range=(1, 300))
    attr = rng.integers(1, 5, size=wl.n_branches).astype(np.int32)
    from paper_2604_26209_amd import binding as B
    for paper in (False, True):
        kw = dict(pos_mode=B.HPD_POS_PAPER_GAP, attr_len=attr, mask_mode=B.HPD_MASK_PAPER) if paper else {}
        okw = dict(pos_mode="paper_gap", attr_len=attr, mask_mode="paper") if paper else {}
        for mode in (3, 4):
            _say(f"G={g} Hkv={hkv} T={wl.max_new} branches={wl.n_branches} literal={paper} mode {mode}")
            a = H.run_hip(wl, kernel_mode=mode, fused=True, **kw)
            H.check_all(wl, a, label=f"g{g}_m{mode}", **okw)
            b = H.run_hip(wl, inputs=a["inputs"], kernel_mode=mode, fused=False, **kw)
            for x, y in zip(a["out"], b["out"]):
                assert torch.equal(x, y)
            _check_prefill(wl, mode, f"g{g}_prefill_m{mode}", attr_len=attr if paper else None)
        _check_prefill(wl, 0, f"g{g}_prefill_m0", attr_len=attr if paper else None)


@pytest.mark.parametrize("literal", [False, True])
@pytest.mark.parametrize("g", [1, 2, 4, 5, 8])
def test_decode_of_many_rows_per_unit(g, literal):
    """The kernel for launches with many rows per unit: row blocks that do not fill a workgroup, documents of one
    token and around a block of 32 keys, no header, branches that end (live ones that are no run of ids; under the literal mask tails of
    several lengths in a tile), tails of 1 .. 11 positions, fp32 and bf16 outputs, paged tails.  Against the oracle, the
    step call against the two-call sequence and against the other kernel (kernel mode 3: bits that differ tell that the
    default was not that kernel)."""
    from paper_2604_26209_amd import binding as B
    pad = 1 << (g - 1).bit_length()
    hkv, steps = 8, 11
    if literal:
        n = min(256, 9 * 32 // pad + 3) // 3
        per, doc, nbr = [3] * 24, [1, 40, 32] * 24, [n, n + 1, n - 1] * 24
        header = [0, 33, 64, 7] * 6
    else:
        n = 8 * 32 // pad
        per, doc, nbr = [4] * 8, [1, 31, 64, 33] * 8, [n, n + 1, n - 1, 4 * 32 // pad] * 8
        header = [0, 33, 64, 7, 0, 1, 32, 95]
    blen = np.full(sum(nbr), steps)
    blen[5::9] = 3
    blen[7::11] = 8
    attr = (1 + np.arange(sum(nbr)) % 4).astype(np.int32)
    wl = W.make_workload("rows", "bf16", g * hkv, hkv, 128, 500000.0, steps, header, per, doc, nbr, blen)
    kw = dict(pos_mode=B.HPD_POS_PAPER_GAP, attr_len=attr, mask_mode=B.HPD_MASK_PAPER) if literal else {}
    okw = dict(pos_mode="paper_gap", attr_len=attr, mask_mode="paper") if literal else {}
    _say(f"many rows per unit: G={g} literal={literal}, {wl.n_branches} branches")
    a = H.run_hip(wl, fused=True, **kw)
    H.check_all(wl, a, prompts=[0, 1], label=f"rows_g{g}_{literal}", **okw)
    b = H.run_hip(wl, inputs=a["inputs"], **kw)
    c = H.run_hip(wl, inputs=a["inputs"], fused=True, kernel_mode=3, **kw)
    d = H.run_hip(wl, inputs=a["inputs"], fused=True, out_f32=False, **kw)
    other = [not torch.equal(x, z) for x, z in zip(a["out"], c["out"])]
    for x, y, z, w in zip(a["out"], b["out"], c["out"], d["out"]):
        assert torch.equal(x, y)
        assert torch.equal(x.to(torch.bfloat16), w)
        # two roundings of queries and weights to 11 bits: as the bound against the oracle, of outputs of size 1
        assert float((x - z).abs().max()) < H.BF16_TOL * float(x.square().mean().sqrt())
    _say(f"  steps that ran it: {[t for t, o in enumerate(other) if o]}")
    assert all(other[:3] if literal else other)
    # the same bits through a page table
    lay = B.layout_from_workload(wl, out_dtype=B.HPD_OUT_F32, **kw)
    table = torch.from_numpy(np.random.default_rng(g).permutation(2 * wl.n_branches).astype(np.int32).reshape(-1, 2)).cuda()
    B.hpd_set_tail_pages(lay, 8, 2 * wl.n_branches, table)
    inputs = a["inputs"]
    pools = B.alloc_pools(lay)
    B.hpd_prefix_fill(lay, inputs.k_raw, inputs.v_raw, pools[0], pools[1])
    for t in range(steps):
        out = torch.zeros_like(a["out"][t])
        B.hpd_decode_step(lay, t, inputs.q[t], inputs.k_new[t], inputs.v_new[t], *pools, out)
        assert torch.equal(out, a["out"][t]), f"step {t}: paged and contiguous outputs differ"


@pytest.mark.parametrize("literal", [False, True])
@pytest.mark.parametrize("g,of_cus", [(1, 1.5), (2, 2.5), (8, 2.5), (3, 2.5), (8, 5), (1, 5), (2, 5)])
def test_decode_of_many_rows_per_unit_by_workgroups_per_cu(g, of_cus, literal):
    """The kernel for many rows per unit in launches of 1.5 workgroups per CU (two at a time), of 2.5 (three, priorities by
    progress) and of 5 (three); that the plan has them run so, the host test of the layouts says for the same batches.  Documents of one token and around one block, row blocks that do not fill a workgroup, branches that
    end, 21 steps: three chunks of tails, so that every piece of LDS that three workgroups per CU leave a wave holds keys and
    values; pools of NaN.  Oracle, two-call sequence and pages of 8 tokens (the same bits), the other kernel."""
    from paper_2604_26209_amd import binding as B
    pad = 1 << (g - 1).bit_length()
    hkv, steps, n = 8, 21, 8 * 32 // pad  # eight row blocks, the last not always full: two workgroups
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    prompts = int(of_cus * cus / (2 * hkv))
    docs = [1] * prompts if literal else [2] * (prompts // 2)
    header = [[0, 33, 64, 7, 95][i % 5] for i in range(len(docs))]
    doc = [[1, 31, 64, 33, 97, 32][i % 6] for i in range(sum(docs))]
    nbr = [n - i % 3 % 2 for i in range(sum(docs))]
    blen = np.full(sum(nbr), steps)
    blen[5::9] = 14
    blen[7::11] = 18
    attr = (1 + np.arange(sum(nbr)) % 4).astype(np.int32)
    wl = W.make_workload("per_cu", "bf16", g * hkv, hkv, 128, 500000.0, steps, header, docs, doc, nbr, blen)
    kw = dict(pos_mode=B.HPD_POS_PAPER_GAP, attr_len=attr, mask_mode=B.HPD_MASK_PAPER) if literal else {}
    okw = dict(pos_mode="paper_gap", attr_len=attr, mask_mode="paper") if literal else {}
    _say(f"many rows per unit, {of_cus} workgroups per CU: G={g} literal={literal}, {wl.n_branches} branches")
    a = H.run_hip(wl, fused=True, **kw)
    H.check_all(wl, a, prompts=[0, len(docs) - 1], label=f"per_cu_g{g}_{literal}", **okw)
    b = H.run_hip(wl, inputs=a["inputs"], **kw)
    c = H.run_hip(wl, inputs=a["inputs"], fused=True, kernel_mode=3, **kw)
    inputs = a["inputs"]
    lay = B.layout_from_workload(wl, out_dtype=B.HPD_OUT_F32, **kw)
    table = torch.from_numpy(np.random.default_rng(g).permutation(3 * wl.n_branches).astype(np.int32).reshape(-1, 3)).cuda()
    B.hpd_set_tail_pages(lay, 8, 3 * wl.n_branches, table)
    pools = [x.fill_(float("nan")) for x in B.alloc_pools(lay)]
    B.hpd_prefix_fill(lay, inputs.k_raw, inputs.v_raw, pools[0], pools[1])
    ran = []
    for t, (x, y, z) in enumerate(zip(a["out"], b["out"], c["out"])):
        assert torch.equal(x, y), f"step {t}: step call and two calls differ"
        ran.append(not torch.equal(x, z))
        # two roundings of queries and weights to 11 bits, of outputs of size 1
        assert float((x - z).abs().max()) < H.BF16_TOL * float(x.square().mean().sqrt()), f"step {t}"
        out = torch.zeros_like(x)
        B.hpd_decode_step(lay, t, inputs.q[t], inputs.k_new[t], inputs.v_new[t], *pools, out)
        assert torch.equal(out, x), f"step {t}: paged and contiguous outputs differ"
    _say(f"  steps that ran it: {[t for t, r in enumerate(ran) if r]}")
    assert sum(ran) >= 3


@pytest.mark.parametrize("literal", [False, True])
def test_decode_of_many_rows_per_unit_takes_no_longer_through_a_page_table(literal):
    """Steps with a long tail that run the kernel for many rows per unit: the page table's entries are there when a tile is
    requested.  Looked up at that time they made these steps take 1.44 and 1.55 times as long; 1.2 is well above what two
    timings of the same call differ by."""
    from paper_2604_26209_amd import binding as B
    hq, hkv, steps, t, docs, per, doc, n = (32, 8, 24, 20, 64, 1, 20, 64) if literal else (64, 8, 48, 44, 64, 1, 141, 16)
    wl = W.make_workload("rows_pages", "bf16", hq, hkv, 128, 500000.0, steps, [0] * (docs // per), [per] * (docs // per), [doc] * docs,
                         [n] * docs, [steps] * (n * docs))
    kw = dict(pos_mode=B.HPD_POS_PAPER_GAP, attr_len=np.ones(n * docs, np.int32), mask_mode=B.HPD_MASK_PAPER) if literal else {}
    lay = [B.layout_from_workload(wl, **kw) for _ in range(2)]
    pages = steps // 8 * wl.n_branches
    table = torch.randperm(pages, device="cuda").to(torch.int32).view(wl.n_branches, -1).contiguous()
    B.hpd_set_tail_pages(lay[1], 8, pages, table)
    pools = [x.normal_() for x in B.alloc_pools(lay[0])]
    q, k, v = (torch.randn(wl.n_branches, h, 128, device="cuda").bfloat16() for h in (hq, hkv, hkv))
    out = torch.zeros_like(q)
    us = _us_in_turn([lambda x=x: B.hpd_decode_step(x, t, q, k, v, *pools, out) for x in lay])
    _say(f"many rows per unit, literal={literal}: {us[0]:.1f} us, through a page table {us[1]:.1f} us")
    assert us[1] < 1.2 * us[0]


@pytest.mark.parametrize("case,mode", [("wide_units_among_narrow", 3), ("ragged", 4)])
def test_uneven_decode_batches_run_the_faster_kernel(case, mode):
    """Uneven batches, in whose workgroups of the kernel for many rows per unit most waves would have no rows: the default
    takes no longer than the other kernel in the shape that is chosen for such a launch (there 1.12 and 1.14 times as long)."""
    from paper_2604_26209_amd import binding as B
    if case == "ragged":
        hq, per, header, doc, nbr = 32, 1, 505, [30 + i * 457 % 457 for i in range(150)], [7 + i * 13 % 29 for i in range(150)]
    else:
        hq, per, header, doc, nbr = 48, 4, 1278, [1 + i % 12 for i in range(104)], [64 if i % 5 == 0 else 1 + i % 8 for i in range(104)]
    wl = W.make_workload("uneven", "bf16", hq, 8, 128, 500000.0, 4, [header] * (len(doc) // per), [per] * (len(doc) // per), doc, nbr,
                         [4] * sum(nbr))
    lay = [B.layout_from_workload(wl) for _ in range(2)]
    B.hpd_set_kernel_mode(lay[1], mode)
    pools = [x.normal_() for x in B.alloc_pools(lay[0])]
    q, k, v = (torch.randn(wl.n_branches, h, 128, device="cuda").bfloat16() for h in (hq, 8, 8))
    out = torch.zeros_like(q)
    us = _us_in_turn([lambda x=x: B.hpd_decode_step(x, 2, q, k, v, *pools, out) for x in lay])
    _say(f"uneven decode, {case}: {us[0]:.1f} us, the streaming kernel {us[1]:.1f} us")
    assert us[0] < 1.08 * us[1]


@pytest.mark.parametrize("prompts", [24, 48])
@pytest.mark.parametrize("case", ["two_blocks", "header", "names", "names_g2"])
def test_literal_decode_of_many_rows_and_few_shared_blocks(case, prompts):
    """Prompts whose header, document and names are two, three or five blocks of 32 keys: with fewer than four, tail tiles are
    among the first loads and the append comes in front of them.  26 steps: all tail formats, in chunks one to four; pools
    of NaN; branches that end.  384 workgroups, two per CU at a time, and 768, three.  Against the oracle, the two-call sequence, pages
    of 8 to 32 tokens (the same bits), and the other kernel, whose bits differ in every step."""
    from paper_2604_26209_amd import binding as B
    hq, header, n = {"two_blocks": (64, 0, 32), "header": (64, 7, 32), "names": (32, 0, 64), "names_g2": (16, 0, 128)}[case]
    steps = 26
    blen = np.full(prompts * n, steps)
    blen[4::11] = 13
    attr = np.ones(prompts * n, np.int32)
    wl = W.make_workload("few_blocks", "bf16", hq, 8, 128, 500000.0, steps, [header] * prompts, [1] * prompts, [20] * prompts, [n] * prompts, blen)
    kw = dict(pos_mode=B.HPD_POS_PAPER_GAP, attr_len=attr, mask_mode=B.HPD_MASK_PAPER)
    _say(f"literal mask, few shared blocks: {case}, {prompts} prompts")
    a = H.run_hip(wl, fused=True, **kw)
    H.check_all(wl, a, prompts=[0, 31 % prompts], label=case, pos_mode="paper_gap", attr_len=attr, mask_mode="paper")
    b = H.run_hip(wl, inputs=a["inputs"], **kw)
    c = H.run_hip(wl, inputs=a["inputs"], fused=True, kernel_mode=3, **kw)
    for t, (x, y, z) in enumerate(zip(a["out"], b["out"], c["out"])):
        assert torch.equal(x, y), f"step {t}: step call and two calls differ"
        assert not torch.equal(x, z), f"step {t} did not run the kernel for many rows"
        assert float((x - z).abs().max()) < H.BF16_TOL * float(x.square().mean().sqrt())
    for page in (8, 16, 32):
        lay = B.layout_from_workload(wl, out_dtype=B.HPD_OUT_F32, **kw)
        per = -(-steps // page)
        table = torch.from_numpy(np.random.default_rng(page).permutation(per * wl.n_branches).astype(np.int32).reshape(-1, per)).cuda()
        B.hpd_set_tail_pages(lay, page, per * wl.n_branches, table)
        pools = [x.fill_(float("nan")) for x in B.alloc_pools(lay)]
        inputs = a["inputs"]
        B.hpd_prefix_fill(lay, inputs.k_raw, inputs.v_raw, pools[0], pools[1])
        for t in range(steps):
            out = torch.zeros_like(a["out"][t])
            B.hpd_decode_step(lay, t, inputs.q[t], inputs.k_new[t], inputs.v_new[t], *pools, out)
            assert torch.equal(out, a["out"][t]), f"step {t}: pages of {page} and contiguous tails differ"


@pytest.mark.parametrize("page", [16, 32, 64])
def test_block_mask_decode_of_many_rows_through_large_pages(page):
    """Steps of several chunks per page, live branches that are no run of ids: the bits of contiguous tails."""
    from paper_2604_26209_amd import binding as B
    docs, n, steps = 64, 16, 70
    blen = np.full(docs * n, steps)
    blen[5::9] = 30
    wl = W.make_workload("large_pages", "bf16", 64, 8, 128, 500000.0, steps, [33] * docs, [1] * docs, [40] * docs, [n] * docs, blen)
    lay = [B.layout_from_workload(wl, out_dtype=B.HPD_OUT_F32) for _ in range(2)]
    per = -(-steps // page)
    table = torch.randperm(per * wl.n_branches, device="cuda").to(torch.int32).view(-1, per).contiguous()
    B.hpd_set_tail_pages(lay[1], page, per * wl.n_branches, table)
    inputs = H.Inputs(wl, lay[0].n_live(), "cuda")
    pools = [[x.fill_(float("nan")) for x in B.alloc_pools(x)] for x in lay]
    _say(f"block mask, pages of {page}")
    for x, p in zip(lay, pools):
        B.hpd_prefix_fill(x, inputs.k_raw, inputs.v_raw, p[0], p[1])
    for t in range(steps):
        outs = []
        for x, p in zip(lay, pools):
            outs.append(torch.zeros(inputs.q[t].shape, device="cuda"))
            B.hpd_decode_step(x, t, inputs.q[t], inputs.k_new[t], inputs.v_new[t], *p, outs[-1])
        assert bool(torch.isfinite(outs[0]).all()) and torch.equal(*outs), f"step {t}"


@pytest.mark.parametrize("value", [float("nan"), float("inf"), float("-inf")])
@pytest.mark.parametrize("literal", [False, True])
@pytest.mark.parametrize("prompts", [24, 48])
def test_non_finite_values_of_a_branch_in_decode_with_many_rows(prompts, literal, value):
    """One value of one branch at one step.  Literal mask: the outputs that are not finite are those of the generic kernel: rows of
    the branch and of later ones.  Block mask: no rows but those that the streaming kernel has (branches that share a tile
    of 32 keys with it).  All others keep the bits of a run without it.  384 workgroups, two per CU at a time, and 768, three."""
    from paper_2604_26209_amd import binding as B
    n, steps, at = 32, 12, 2
    attr = np.ones(prompts * n, np.int32)
    wl = W.make_workload("non_finite", "bf16", 64, 8, 128, 500000.0, steps, [7] * prompts, [1] * prompts, [40] * prompts, [n] * prompts,
                         np.full(prompts * n, steps))
    kw = dict(pos_mode=B.HPD_POS_PAPER_GAP, attr_len=attr, mask_mode=B.HPD_MASK_PAPER) if literal else {}
    _say(f"non-finite value, literal={literal}, {prompts} prompts: {value}")
    clean = H.run_hip(wl, fused=True, **kw)
    inputs = clean["inputs"]
    inputs.v_new[at][3 * n + 5, 1, 3] = value
    a = H.run_hip(wl, inputs=inputs, fused=True, **kw)
    ref = H.run_hip(wl, inputs=inputs, fused=True, kernel_mode=1 if literal else 3, **kw)
    for t in range(steps):
        bad, may = (~torch.isfinite(x["out"][t]) for x in (a, ref))
        assert bool((bad & ~may).sum() == 0) and torch.equal(a["out"][t][~bad], clean["out"][t][~bad]), f"step {t}"
        assert bool(bad[3 * n + 5].any()) == (t >= at) and (not literal or torch.equal(bad, may)), f"step {t}"


def _set_score_range(inp, case):
    bf = lambda x: x.float().to(torch.bfloat16)
    if case in ("peaked_x4", "argmax_x16", "flat_div16"):
        inp.q = [bf(x.float() * dict(peaked_x4=4.0, argmax_x16=16.0, flat_div16=1.0 / 16)[case]) for x in inp.q]
    elif case == "rising":
        n = inp.k_raw.shape[0]
        inp.k_raw = bf(inp.k_raw.float() + torch.arange(n, device="cuda")[:, None, None] % 500 * (4.0 / 500))
        inp.k_new = [bf(x.float() + 4.0 + 0.3 * t) for t, x in enumerate(inp.k_new)]
        inp.q = [bf(x.float() * 0.5 + 1.0) for x in inp.q]
    else:
        sign = 1.0 if case == "common_offset" else -1.0
        inp.q = [bf(x.float() + 1.0) for x in inp.q]
        inp.k_raw = bf(inp.k_raw.float() + sign)
        inp.k_new = [bf(x.float() + sign) for x in inp.k_new]


@pytest.mark.parametrize("case", ["peaked_x4", "argmax_x16", "flat_div16", "common_offset", "negative_offset", "rising"])
def test_score_ranges_of_decode_with_many_rows_per_unit(case):
    """The inputs of test_score_ranges_of_the_online_softmax, and scores all near -16, for the kernel for many rows per
    unit: against the oracle, and against the other kernel, whose bits differ.  That one rounds the same queries to the same
    halves, so what is left are the weights' 11 bits: 2^-11 of a value, which is below 6.  Scores 16 times as wide are
    compared with the other kernel only: there a query's 11 bits move a score of 60 by up to 60 * 2^-12, and of two keys that
    tie each one's weight by a quarter of that, 2e-2 between values 5 apart, in some of these 65 536 rows (0.0213 x RMS in
    either kernel, 2e-5 in the generic one, which keeps the query in fp32)."""
    from paper_2604_26209_amd import binding as B
    wl = W.make_workload("rows_ranges", "bf16", 32, 4, 128, 500000.0, 4, [40] * 16, [4] * 16, [50, 200, 97, 33] * 16, [32] * 64,
                         [4] * 2048)
    lay = B.layout_from_workload(wl)
    inp = H.Inputs(wl, lay.n_live(), "cuda", lay.counts()[B.HPD_C_N_PREFIX_TOKENS])
    _set_score_range(inp, case)
    _say(f"score ranges, many rows: {case}")
    a = H.run_hip(wl, inputs=inp, fused=True)
    if case != "argmax_x16":
        H.check_all(wl, a, prompts=[0, 5], label=f"rows_{case}")
    c = H.run_hip(wl, inputs=inp, fused=True, kernel_mode=3)
    assert any(not torch.equal(x, z) for x, z in zip(a["out"], c["out"]))
    assert all(float((x - z).abs().max()) < 6 * 2.0 ** -11 for x, z in zip(a["out"], c["out"]))


@pytest.mark.parametrize("case", ["peaked_x4", "argmax_x16", "flat_div16", "common_offset", "negative_offset", "rising"])
def test_score_ranges_of_literal_decode_with_many_rows_per_unit(case):
    """The same under the literal mask, with tails of one and two chunks, and with the same bounds."""
    from paper_2604_26209_amd import binding as B
    prompts, n, steps = 48, 32, 12
    attr = np.ones(prompts * n, np.int32)
    wl = W.make_workload("rows_ranges", "bf16", 64, 8, 128, 500000.0, steps, [40] * prompts, [1] * prompts, [97] * prompts, [n] * prompts,
                         [steps] * (prompts * n))
    kw = dict(pos_mode=B.HPD_POS_PAPER_GAP, attr_len=attr, mask_mode=B.HPD_MASK_PAPER)
    lay = B.layout_from_workload(wl, **kw)
    inp = H.Inputs(wl, lay.n_live(), "cuda", lay.counts()[B.HPD_C_N_PREFIX_TOKENS])
    _set_score_range(inp, case)
    _say(f"score ranges, many rows, literal mask: {case}")
    a = H.run_hip(wl, inputs=inp, fused=True, **kw)
    if case != "argmax_x16":
        H.check_all(wl, a, prompts=[0, 5], label=f"rows_{case}", pos_mode="paper_gap", attr_len=attr, mask_mode="paper")
    c = H.run_hip(wl, inputs=inp, fused=True, kernel_mode=3, **kw)
    assert all(not torch.equal(x, z) for x, z in zip(a["out"], c["out"]))
    assert all(float((x - z).abs().max()) < 6 * 2.0 ** -11 for x, z in zip(a["out"], c["out"]))


@pytest.mark.parametrize("seed,kw", [(120, dict(hq=8, hkv=2, p=3, j_range=(1, 4), n_range=(1, 14), l_range=(1, 200))),
                                     (121, dict(hq=8, hkv=8, p=2, j_range=(2, 3), n_range=(3, 40), l_range=(1, 90))),
                                     (122, dict(hq=16, hkv=2, p=2, j_range=(1, 2), n_range=(1, 30), l_range=(30, 300)))])
def test_device_side_pruning_equals_host_lists(seed, kw):
    """hpd_dynamic_*: the live list is built on the GPU from per-row "finished" flags (here: a
    branch is flagged in the step that exhausts its length).  The device-side live list and
    count must equal the layout's host-built lists of every step, and hpd_dynamic_step must
    write the very bits hpd_decode_step writes."""
    from paper_2604_26209_amd import binding as B
    wl = W.random_workload(seed, dtype="bf16", d=128, base=500000.0, t=10, h_range=(0, 70), **kw)
    ref = H.run_hip(wl, fused=True)
    lay = B.layout_from_workload(wl, out_dtype=B.HPD_OUT_F32)
    inputs = ref["inputs"]
    kp, vp, kt, vt = B.alloc_pools(lay)
    for x in (kp, vp, kt, vt):
        x.fill_(float("nan"))
    B.hpd_prefix_fill(lay, inputs.k_raw, inputs.v_raw, kp, vp)
    B.hpd_dynamic_begin(lay)
    live_ptr, n_ptr = B.hpd_dynamic_state(lay)
    assert live_ptr != 0 and n_ptr != 0
    n_live = lay.n_live()
    live_flat = B.hpd_layout_query(lay, B.HPD_Q_LIVE_BRANCH)
    off = 0
    for t in range(wl.max_new):
        n = int(n_live[t])
        want_live = live_flat[off:off + n]
        off += n
        got_n, got_live = B.hpd_dynamic_read(lay, wl.n_branches)
        assert got_n == n, f"step {t}: n_live {got_n} != {n}"
        assert np.array_equal(got_live, want_live), f"step {t}: live list differs"
        out = torch.full((max(n, 1), wl.n_q_heads, wl.head_dim), float("nan"), dtype=torch.float32, device="cuda")
        if n:
            B.hpd_dynamic_step(lay, t, inputs.q[t], inputs.k_new[t], inputs.v_new[t], kp, vp, kt, vt, out)
            assert torch.equal(out[:n], ref["out"][t]), f"step {t}: outputs differ from hpd_decode_step"
        if t + 1 < wl.max_new:
            fin = torch.from_numpy((wl.branch_len[want_live] == t + 1).astype(np.uint8)).cuda() if n else \
                torch.zeros(1, dtype=torch.uint8, device="cuda")
            B.hpd_dynamic_prune(lay, fin)
    with pytest.raises(B.HpdError):
        B.hpd_dynamic_step(lay, 0, inputs.q[0], inputs.k_new[0], inputs.v_new[0], kp, vp, kt, vt, out)  # wrong step


@pytest.mark.parametrize("literal", [False, True])
@pytest.mark.parametrize("seed", [130, 131])
def test_device_side_pruning_with_lengths_unknown_to_the_layout(seed, literal):
    """The use the entry points exist for: the layout is built with every branch at the full
    step budget (nobody knows yet where a branch ends), and branches leave when the caller
    flags them (the stop condition of Section 4.3.4).  With flags taken from a hidden
    length per branch, every step must match the oracle run on the workload that has those
    lengths.  Under the literal mask a branch that has left stays visible to the later ones
    as far as it got: the device keeps the number of tokens it reached."""
    import dataclasses
    from paper_2604_26209_amd import binding as B
    wl = W.random_workload(seed, dtype="bf16", d=128, base=500000.0, t=9, hq=8, hkv=2, p=3,
                           j_range=(1, 3), n_range=(1, 20), l_range=(1, 260), h_range=(0, 50))
    cap = dataclasses.replace(wl, branch_len=np.full(wl.n_branches, wl.max_new, dtype=np.int32))
    attr = np.random.default_rng(seed).integers(1, 5, size=wl.n_branches).astype(np.int32)
    kw = dict(pos_mode=B.HPD_POS_PAPER_GAP, attr_len=attr, mask_mode=B.HPD_MASK_PAPER) if literal else {}
    okw = dict(pos_mode="paper_gap", attr_len=attr, mask_mode="paper") if literal else {}
    ref = H.run_hip(wl, fused=True, **kw)  # for the inputs, positions and slots of the hidden lengths
    inputs = ref["inputs"]
    lay = B.layout_from_workload(cap, out_dtype=B.HPD_OUT_F32, **kw)
    kp, vp, kt, vt = B.alloc_pools(lay)
    B.hpd_prefix_fill(lay, inputs.k_raw, inputs.v_raw, kp, vp)
    B.hpd_dynamic_begin(lay)
    outs = []
    for t in range(wl.max_new):
        live = np.nonzero(wl.branch_len > t)[0]
        got_n, got_live = B.hpd_dynamic_read(lay, wl.n_branches)
        assert got_n == len(live) and np.array_equal(got_live, live), f"step {t}: live list differs"
        out = torch.full((max(len(live), 1), wl.n_q_heads, wl.head_dim), float("nan"), dtype=torch.float32,
                         device="cuda")
        if len(live):
            B.hpd_dynamic_step(lay, t, inputs.q[t], inputs.k_new[t], inputs.v_new[t], kp, vp, kt, vt, out)
        outs.append(out[:len(live)])
        if t + 1 < wl.max_new:
            fin = (wl.branch_len[live] == t + 1).astype(np.uint8) if len(live) else np.zeros(1, np.uint8)
            B.hpd_dynamic_prune(lay, torch.from_numpy(fin).cuda())
    hip = dict(ref)
    hip["out"] = outs
    H.check_all(wl, hip, label=f"dynamic_{seed}", **okw)


class _PageAllocator:
    """Host-side page allocator of the paged-tail tests: pages come from a shuffled free list,
    a branch takes one when it reaches a page boundary and gives all of them back when it
    ends, so pages are reused and hold stale rows of other branches."""

    def __init__(self, wl, page_size, seed):
        self.wl, self.ps = wl, page_size
        self.ppb = -(-wl.max_new // page_size)
        need, held = 0, 0
        for t in range(wl.max_new):  # pages in use at the same time
            if t % page_size == 0:
                held += int((wl.branch_len > t).sum())
            need = max(need, held)
            held -= int(((wl.branch_len == t + 1) * (-(-(t + 1) // page_size))).sum())
        self.n_pages = max(need, 1)
        self.free = list(np.random.default_rng(seed).permutation(self.n_pages))
        self.table = np.full((wl.n_branches, self.ppb), -7, dtype=np.int32)  # -7: never assigned

    def before_step(self, t):
        if t % self.ps == 0:
            for b in np.nonzero(self.wl.branch_len > t)[0]:
                self.table[b, t // self.ps] = self.free.pop()

    def after_step(self, t):
        for b in np.nonzero(self.wl.branch_len == t + 1)[0]:
            for i in range(self.ppb):
                if self.table[b, i] >= 0:
                    self.free.append(int(self.table[b, i]))
                    self.table[b, i] = -7

    def slots(self, live, t):
        return self.table[live, t // self.ps].astype(np.int64) * self.ps + t % self.ps


@pytest.mark.parametrize("case", ["stream_fused", "stream_two_call", "f32", "generic_f32", "dynamic"])
def test_paged_tails(case):
    """hpd_set_tail_pages: tail pools of n_pages pages (fewer than B * T slots; pages of ended
    branches are reused) against the contiguous pools: same outputs bit for bit, slots as the
    page table says, and within tolerance of the oracle."""
    from paper_2604_26209_amd import binding as B
    _say(f"paged tails: {case}")
    f32 = case in ("f32", "generic_f32")  # the fp32 kernel, the generic one
    mode = 1 if case == "generic_f32" else 0
    if f32:
        wl = W.random_workload(140, dtype="f32", hq=4, hkv=2, d=64, t=19, p=2, n_range=(1, 9))
    else:
        wl = W.random_workload(141, dtype="bf16", hq=8, hkv=2, d=128, base=500000.0, t=21, p=3,
                               j_range=(1, 3), n_range=(1, 14), h_range=(0, 80), l_range=(1, 200))
    ps = 8
    ref = H.run_hip(wl, fused=(case != "stream_two_call"), kernel_mode=mode)
    inputs = ref["inputs"]
    lay = B.layout_from_workload(wl, out_dtype=B.HPD_OUT_SAME if f32 else B.HPD_OUT_F32)
    B.hpd_set_kernel_mode(lay, mode)
    alloc = _PageAllocator(wl, ps, seed=7)
    assert alloc.n_pages * ps < wl.n_branches * wl.max_new, "the case must save memory"
    table = torch.from_numpy(alloc.table).cuda()
    full = B.hpd_layout_query(lay, B.HPD_Q_POOL_BYTES)
    B.hpd_set_tail_pages(lay, ps, alloc.n_pages, table)
    paged = B.hpd_layout_query(lay, B.HPD_Q_POOL_BYTES)
    assert paged[2] * wl.n_branches * wl.max_new == full[2] * alloc.n_pages * ps and paged[0] == full[0]
    kp, vp, kt, vt = B.alloc_pools(lay)
    for x in (kp, vp, kt, vt):
        x.fill_(float("nan"))
    B.hpd_prefix_fill(lay, inputs.k_raw, inputs.v_raw, kp, vp)
    if case == "dynamic":
        B.hpd_dynamic_begin(lay)
    outs = []
    for t in range(wl.max_new):
        live = np.nonzero(wl.branch_len > t)[0]
        n = len(live)
        alloc.before_step(t)
        table.copy_(torch.from_numpy(alloc.table))
        out = torch.full((n, wl.n_q_heads, wl.head_dim), float("nan"), dtype=torch.float32, device="cuda")
        slot = torch.full((max(n, 1),), -1, dtype=torch.int64, device="cuda")
        if n:
            a = (lay, t, inputs.q[t], inputs.k_new[t], inputs.v_new[t], kp, vp, kt, vt, out)
            if case == "dynamic":
                B.hpd_dynamic_step(*a)
            elif case == "stream_two_call":
                B.hpd_kv_append(lay, t, inputs.k_new[t], inputs.v_new[t], kt, vt, slot)
                B.hpd_decode_attention(lay, t, inputs.q[t], kp, vp, kt, vt, out)
                assert np.array_equal(slot[:n].cpu().numpy(), alloc.slots(live, t)), f"step {t}: slots"
            else:
                B.hpd_decode_step(*a)
            assert torch.equal(out, ref["out"][t]), f"step {t}: paged and contiguous outputs differ"
        outs.append(out)
        if case == "dynamic" and t + 1 < wl.max_new:
            fin = (wl.branch_len[live] == t + 1).astype(np.uint8) if n else np.zeros(1, np.uint8)
            B.hpd_dynamic_prune(lay, torch.from_numpy(fin).cuda())
        torch.cuda.synchronize()  # the table is rewritten on the host for the next step
        alloc.after_step(t)
    hip = dict(ref)
    hip["out"] = outs
    H.check_all(wl, hip, label=f"paged_{case}")
    # switching paging off restores the contiguous sizes; bad arguments are refused
    B.hpd_set_tail_pages(lay, 0)
    assert np.array_equal(B.hpd_layout_query(lay, B.HPD_Q_POOL_BYTES), full)
    for bad in (4, 12, -8):
        with pytest.raises(B.HpdError):
            B.hpd_set_tail_pages(lay, bad, 4, table)
    with pytest.raises(B.HpdError):
        B.hpd_set_tail_pages(lay, 8, 0, table)
    with pytest.raises(B.HpdError):
        B.hpd_set_tail_pages(lay, 8, 4, None)


@pytest.mark.parametrize("seed", range(150, 158))
def test_paged_tails_random_sweep(seed):
    """Page size, group size, workgroup shape, step budget and batch drawn from the seed: the
    paged step call against the contiguous one, bit for bit.  Odd seeds use the device-side
    lists, whose launches split a document's rows by its full branch count (the host does not
    know the live count), so sums may be grouped differently than in hpd_decode_step: those
    are checked against the oracle."""
    from paper_2604_26209_amd import binding as B
    rng = np.random.default_rng(seed)
    g = (1, 2, 4, 8)[seed % 4]
    hkv = int(rng.choice([1, 2]))
    ps = (8, 16, 32)[seed % 3]
    t_max = int(rng.integers(2, 41))
    mode = 3 + (seed // 2) % 2
    wl = W.random_workload(seed, dtype="bf16", hq=hkv * g, hkv=hkv, d=128, base=500000.0, t=t_max,
                           p=int(rng.integers(1, 4)), j_range=(1, 3), n_range=(1, int(rng.integers(2, 30))),
                           h_range=(0, 60), l_range=(1, int(rng.integers(2, 300))))
    _say(f"paged sweep seed {seed}: G={g} Hkv={hkv} T={t_max} page {ps} mode {mode} branches {wl.n_branches}")
    ref = H.run_hip(wl, kernel_mode=mode, fused=True)
    inputs = ref["inputs"]
    lay = B.layout_from_workload(wl, out_dtype=B.HPD_OUT_F32)
    B.hpd_set_kernel_mode(lay, mode)
    alloc = _PageAllocator(wl, ps, seed=seed)
    table = torch.from_numpy(alloc.table).cuda()
    B.hpd_set_tail_pages(lay, ps, alloc.n_pages, table)
    kp, vp, kt, vt = B.alloc_pools(lay)
    for x in (kp, vp, kt, vt):
        x.fill_(float("nan"))
    B.hpd_prefix_fill(lay, inputs.k_raw, inputs.v_raw, kp, vp)
    dynamic = seed % 2 == 1
    if dynamic:
        B.hpd_dynamic_begin(lay)
    outs = []
    for t in range(wl.max_new):
        live = np.nonzero(wl.branch_len > t)[0]
        if len(live) == 0:
            break
        alloc.before_step(t)
        table.copy_(torch.from_numpy(alloc.table))
        out = torch.full((len(live), wl.n_q_heads, wl.head_dim), float("nan"), dtype=torch.float32, device="cuda")
        a = (lay, t, inputs.q[t], inputs.k_new[t], inputs.v_new[t], kp, vp, kt, vt, out)
        (B.hpd_dynamic_step if dynamic else B.hpd_decode_step)(*a)
        if not dynamic:
            assert torch.equal(out, ref["out"][t]), f"seed {seed} step {t}: paged and contiguous outputs differ"
        outs.append(out)
        if dynamic and t + 1 < wl.max_new:
            B.hpd_dynamic_prune(lay, torch.from_numpy((wl.branch_len[live] == t + 1).astype(np.uint8)).cuda())
        torch.cuda.synchronize()
        alloc.after_step(t)
    while len(outs) < wl.max_new:
        outs.append(torch.zeros((0, wl.n_q_heads, wl.head_dim), dtype=torch.float32, device="cuda"))
    hip = dict(ref)
    hip["out"] = outs
    H.check_all(wl, hip, label=f"paged_sweep_{seed}")


@pytest.mark.parametrize("dynamic", [False, True])
def test_decode_pass_replayed_from_a_hip_graph(dynamic):
    """The step calls only enqueue kernels (no allocation, no synchronisation, no memset), so a
    whole decode pass can be captured in a HIP graph.  The graph is replayed three times, with
    eager work and synchronisations in between (tails cleared, outputs poisoned), and every
    replay must reproduce the eager pass bit for bit."""
    from paper_2604_26209_amd import binding as B
    wl = W.random_workload(180, dtype="bf16", hq=8, hkv=2, d=128, base=500000.0, t=9, p=3,
                           j_range=(1, 3), n_range=(1, 10), h_range=(0, 60), l_range=(1, 150))
    ref = H.run_hip(wl, fused=True)
    inputs = ref["inputs"]
    lay = B.layout_from_workload(wl, out_dtype=B.HPD_OUT_F32)
    kp, vp, kt, vt = B.alloc_pools(lay)
    kp.zero_(), vp.zero_()
    B.hpd_prefix_fill(lay, inputs.k_raw, inputs.v_raw, kp, vp)
    n_live = lay.n_live()
    outs = [torch.zeros((int(n_live[t]), wl.n_q_heads, wl.head_dim), dtype=torch.float32, device="cuda")
            for t in range(wl.max_new)]
    fins = [torch.from_numpy((wl.branch_len[np.nonzero(wl.branch_len > t)[0]] == t + 1).astype(np.uint8)).cuda()
            for t in range(wl.max_new)]

    def one_pass():
        if dynamic:
            B.hpd_dynamic_begin(lay)
        for t in range(wl.max_new):
            if int(n_live[t]) == 0:
                break
            a = (lay, t, inputs.q[t], inputs.k_new[t], inputs.v_new[t], kp, vp, kt, vt, outs[t])
            (B.hpd_dynamic_step if dynamic else B.hpd_decode_step)(*a)
            if dynamic and t + 1 < wl.max_new and int(n_live[t + 1]) > 0:
                B.hpd_dynamic_prune(lay, fins[t])

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        one_pass()  # also the first hpd_dynamic_begin, which allocates and synchronises
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        one_pass()
    for rep in range(3):
        kt.fill_(float("nan")), vt.fill_(float("nan"))
        for o in outs:
            o.fill_(float("nan"))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        for t in range(wl.max_new):
            assert torch.equal(outs[t], ref["out"][t]), f"replay {rep} step {t}: differs from the eager pass"


@pytest.mark.parametrize("dynamic", [False, True])
def test_paged_tails_under_the_literal_mask(dynamic):
    """Under HPD_MASK_PAPER a branch that has left is still read by the later branches of its
    prompt, so its pages stay; the pools still hold only the pages that were ever reached.
    Paged step calls (host lists / device-side lists) against the contiguous ones."""
    from paper_2604_26209_amd import binding as B
    wl = W.random_workload(143 + int(dynamic), dtype="bf16", hq=8, hkv=2, d=128, base=500000.0, t=20, p=3,
                           j_range=(1, 3), n_range=(1, 12), h_range=(0, 60), l_range=(1, 150))
    attr = np.random.default_rng(143).integers(1, 5, size=wl.n_branches).astype(np.int32)
    kw = dict(pos_mode=B.HPD_POS_PAPER_GAP, attr_len=attr, mask_mode=B.HPD_MASK_PAPER)
    ref = H.run_hip(wl, fused=True, **kw)
    inputs = ref["inputs"]
    lay = B.layout_from_workload(wl, out_dtype=B.HPD_OUT_F32, **kw)
    ps = 8
    ppb = -(-wl.max_new // ps)
    need = int(np.sum(-(-wl.branch_len // ps)))  # pages ever reached
    assert need < wl.n_branches * ppb
    order = list(np.random.default_rng(5).permutation(need))
    table_h = np.full((wl.n_branches, ppb), -7, dtype=np.int32)
    table = torch.from_numpy(table_h).cuda()
    B.hpd_set_tail_pages(lay, ps, need, table)
    kp, vp, kt, vt = B.alloc_pools(lay)
    for x in (kp, vp, kt, vt):
        x.fill_(float("nan"))
    B.hpd_prefix_fill(lay, inputs.k_raw, inputs.v_raw, kp, vp)
    if dynamic:
        B.hpd_dynamic_begin(lay)
    outs = []
    for t in range(wl.max_new):
        live = np.nonzero(wl.branch_len > t)[0]
        if t % ps == 0:
            for b in live:
                table_h[b, t // ps] = order.pop()
            table.copy_(torch.from_numpy(table_h))
        out = torch.full((len(live), wl.n_q_heads, wl.head_dim), float("nan"), dtype=torch.float32, device="cuda")
        if len(live):
            a = (lay, t, inputs.q[t], inputs.k_new[t], inputs.v_new[t], kp, vp, kt, vt, out)
            (B.hpd_dynamic_step if dynamic else B.hpd_decode_step)(*a)
            if not dynamic:
                assert torch.equal(out, ref["out"][t]), f"step {t}: paged and contiguous outputs differ"
        outs.append(out)
        if dynamic and t + 1 < wl.max_new:
            fin = (wl.branch_len[live] == t + 1).astype(np.uint8) if len(live) else np.zeros(1, np.uint8)
            B.hpd_dynamic_prune(lay, torch.from_numpy(fin).cuda())
        torch.cuda.synchronize()
    assert not order
    hip = dict(ref)
    hip["out"] = outs
    H.check_all(wl, hip, label="paged_literal", pos_mode="paper_gap", attr_len=attr, mask_mode="paper")


def test_bf16_output_is_the_fp32_output_rounded_once():
    """out_dtype = SAME writes RNE(bf16) of exactly the values out_dtype = F32 writes."""
    _say("bf16 out == rne(fp32 out)")
    wl = W.config(2, n_prompts=3)
    for mode in (1, 3, 4):
        a = H.run_hip(wl, kernel_mode=mode, out_f32=True)
        b = H.run_hip(wl, inputs=a["inputs"], kernel_mode=mode, out_f32=False)
        for x, y in zip(a["out"], b["out"]):
            assert y.dtype == torch.bfloat16 and torch.equal(x.to(torch.bfloat16), y)


def test_mfma_edge_shapes():
    cases = {
        "single_branch_h0_l1": W.make_workload("e1", "bf16", 4, 1, 128, 500000.0, 3, [0], [1], [1], [1]),
        "mha_g1": W.make_workload("e2", "bf16", 2, 2, 128, 500000.0, 2, [5], [1], [33], [3]),
        "many_rows_two_row_groups": W.make_workload("e3", "bf16", 16, 2, 128, 500000.0, 2, [40], [1],
                                                    [100], [40]),  # 8*40 = 320 rows -> 10 blocks
        "exact_blocks": W.make_workload("e4", "bf16", 8, 2, 128, 500000.0, 4, [64], [2], [128, 96], [8, 16]),
        "t1": W.make_workload("e5", "bf16", 8, 8, 128, 500000.0, 1, [7], [1], [9], [5]),
        "long_tail": W.make_workload("e6", "bf16", 8, 2, 128, 500000.0, 40, [33], [1], [70], [9]),
        "nine_row_blocks": W.make_workload("e7", "bf16", 8, 1, 128, 500000.0, 2, [10], [2], [50, 45], [35, 3]),
    }
    for name, wl in cases.items():
        for mode in (3, 4):
            for fused in (False, True):
                _say(f"mfma edge {name} mode {mode} fused {fused}")
                hip = H.run_hip(wl, kernel_mode=mode, fused=fused)
                H.check_all(wl, hip, label=name)


def test_paper_gap_positions_mode():
    _say("paper-gap mode")
    wl = W.random_workload(21, dtype="bf16", hq=8, hkv=2, d=128, base=500000.0, t=4, p=2)
    attr = np.random.default_rng(3).integers(1, 6, size=wl.n_branches).astype(np.int32)
    for mode, fused in ((3, False), (3, True), (4, False), (4, True)):  # wide / narrow workgroup shape
        hip = H.run_hip(wl, pos_mode=1, attr_len=attr, kernel_mode=mode, fused=fused)
        H.check_all(wl, hip, pos_mode="paper_gap", attr_len=attr, label=f"gap_m{mode}")
    wl = W.random_workload(22, dtype="f32", t=4, p=2)
    attr = np.random.default_rng(4).integers(1, 6, size=wl.n_branches).astype(np.int32)
    hip = H.run_hip(wl, pos_mode=1, attr_len=attr)
    H.check_all(wl, hip, pos_mode="paper_gap", attr_len=attr, label="gap_f32")


def test_paper_literal_mask_mode():
    """HPD_MASK_PAPER: one causal order by position ID over the whole stacked prompt (all
    documents, the tokens of every earlier branch up to the current step, finished ones
    included).  Outputs against the oracle's dense mask, and the exported mask bit-exact."""
    from paper_2604_26209_amd import binding as B
    cases = [("f32", dict(hq=4, hkv=2, d=64, t=5, p=2, j_range=(1, 3), n_range=(1, 5), l_range=(1, 40)), (1,)),
             ("bf16", dict(hq=8, hkv=2, d=128, base=500000.0, t=6, p=3, j_range=(1, 4), n_range=(1, 9),
                           h_range=(0, 70), l_range=(1, 150)), (1, 3, 4))]
    for i, (dt, kw, modes) in enumerate(cases):
        wl = W.random_workload(70 + i, dtype=dt, **kw)
        attr = np.random.default_rng(70 + i).integers(1, 6, size=wl.n_branches).astype(np.int32)
        for mode in modes:
            for fused in (False, True):
                _say(f"paper mask {dt} mode {mode} fused {fused}")
                hip = H.run_hip(wl, pos_mode=1, attr_len=attr, mask_mode=B.HPD_MASK_PAPER, fused=fused,
                                kernel_mode=mode)
                H.check_all(wl, hip, pos_mode="paper_gap", attr_len=attr, mask_mode="paper",
                            label=f"paper_{dt}_m{mode}")
        orc, _ = H.run_oracle(wl, hip["inputs"], pos_mode="paper_gap", attr_len=attr, mask_mode="paper")
        for p, po in orc.prompts.items():
            s = B.hpd_expand_mask(hip["layout"], p, wl.max_new - 1)
            m = torch.full((s, s), 7, dtype=torch.uint8, device="cuda")
            B.hpd_expand_mask(hip["layout"], p, wl.max_new - 1, m)
            assert np.array_equal(m.cpu().numpy(), po.dense_mask())
    # the literal mask orders a prompt by position ID: positions that restart per document do not
    with pytest.raises(B.HpdError):
        B.layout_from_workload(wl, pos_mode=0, mask_mode=B.HPD_MASK_PAPER)


@pytest.mark.parametrize("g", [1, 2, 4, 8])
def test_paper_literal_mask_stream_kernel_shapes(g):
    """The streaming kernel under HPD_MASK_PAPER: every group size, all workgroup shapes,
    prompts with more rows than one workgroup takes (several row groups, each appending the
    earlier groups' newest tokens itself in the step call), finished branches as keys, a tail
    of more than one chunk of 8 positions; the step call equals the two-call sequence bit for
    bit."""
    from paper_2604_26209_amd import binding as B
    wl = W.random_workload(80 + g, dtype="bf16", hq=8, hkv=8 // g, d=128, base=500000.0, t=11, p=2,
                           j_range=(2, 4), n_range=(3, 30 if g < 4 else 20), h_range=(0, 90), l_range=(1, 200))
    attr = np.random.default_rng(80 + g).integers(1, 4, size=wl.n_branches).astype(np.int32)
    for mode in (3, 4):
        _say(f"paper mask stream G={g} mode {mode}: {wl.n_branches} branches")
        a = H.run_hip(wl, pos_mode=1, attr_len=attr, mask_mode=B.HPD_MASK_PAPER, kernel_mode=mode,
                      fused=False, poison_pools=True)
        rel = H.check_all(wl, a, pos_mode="paper_gap", attr_len=attr, mask_mode="paper", label=f"paper_g{g}_m{mode}")
        _say(f"  worst err/rms {rel:.2e}")
        b = H.run_hip(wl, inputs=a["inputs"], pos_mode=1, attr_len=attr, mask_mode=B.HPD_MASK_PAPER,
                      kernel_mode=mode, fused=True, poison_pools=True)
        for x, y in zip(a["out"], b["out"]):
            assert torch.equal(x, y)


def _check_prefill(wl, mode, label, out_f32=None, attr_len=None, change=None):
    """hpd_prefill_attention against the oracle's prefill_attention, all prompts.  With
    `attr_len`: the literal mask (gap positions), whose prefix also holds the attribute names.
    `change` maps (queries, keys) to the ones used."""
    from paper_2604_26209_amd import binding as B
    if out_f32 is None:
        out_f32 = wl.dtype == "bf16"
    paper = attr_len is not None
    layout = B.layout_from_workload(wl, out_dtype=B.HPD_OUT_F32 if out_f32 else B.HPD_OUT_SAME,
                                    **(dict(pos_mode=B.HPD_POS_PAPER_GAP, attr_len=attr_len,
                                            mask_mode=B.HPD_MASK_PAPER) if paper else {}))
    if mode:
        B.hpd_set_kernel_mode(layout, mode)
    n_tok = int(layout.counts()[B.HPD_C_N_PREFIX_TOKENS])
    assert n_tok == wl.n_prefix_tokens + (int(np.sum(attr_len)) if paper else 0)
    inputs = H.Inputs(wl, layout.n_live(), "cuda", n_tok)
    q = W.normal_values((n_tok, wl.n_q_heads, wl.head_dim), wl.value_seed * 1000 + 3, "cuda", wl.dtype)
    if change:
        q, inputs.k_raw = change(q, inputs.k_raw)
    kp, vp, kt, vt = B.alloc_pools(layout)
    for x in (kp, vp):
        x.fill_(float("nan"))
    B.hpd_prefix_fill(layout, inputs.k_raw, inputs.v_raw, kp, vp)
    out = torch.full((n_tok, wl.n_q_heads, wl.head_dim), float("nan"),
                     dtype=torch.float32 if out_f32 else H.torch_dtype(wl), device="cuda")
    B.hpd_prefill_attention(layout, q, kp, vp, out)
    torch.cuda.synchronize()
    orc, _ = H.run_oracle(wl, inputs, steps=[], **(dict(pos_mode="paper_gap", attr_len=attr_len,
                                                        mask_mode="paper") if paper else {}))
    ref = orc.prefill_attention(q.float().cpu().numpy())
    got = out.float().cpu().numpy()
    assert np.isfinite(got).all(), f"{label}: non-finite output"
    worst = 0.0
    for p, want in ref.items():
        a0, a1 = orc.prefix_range[p]
        err = float(np.abs(got[a0:a1] - want).max())
        if wl.dtype == "f32":
            assert err <= H.F32_TOL, f"{label} prompt {p}: max-abs {err:.3e}"
            worst = max(worst, err)
        else:
            # The RMS of a token's outputs falls from |v| (a token that sees one key) to
            # |v| / sqrt(keys): the bound is taken per token, relative to that token's own
            # RMS over its Hq x D outputs.
            diff = np.abs(got[a0:a1] - want).reshape(a1 - a0, -1).max(axis=1)
            rms = np.sqrt(np.mean(want.astype(np.float64).reshape(a1 - a0, -1) ** 2, axis=1))
            bad = np.nonzero(diff > H.BF16_TOL * rms)[0]
            assert bad.size == 0, (f"{label} prompt {p}: token {bad[0]} max-abs {diff[bad[0]]:.3e} > "
                                   f"{H.BF16_TOL} * rms {rms[bad[0]]:.3e}")
            worst = max(worst, float((diff / rms).max()))
    return worst


def test_prefill_attention_fp32_generic():
    for seed, kw in [(90, dict(hq=4, hkv=2, d=64, t=2, p=3, j_range=(1, 3), h_range=(0, 20), l_range=(1, 70))),
                     (91, dict(hq=2, hkv=2, d=32, t=1, p=2, h_range=(0, 0), l_range=(1, 5)))]:
        wl = W.random_workload(seed, dtype="f32", **kw)
        _say(f"prefill f32 seed {seed}: {wl.n_prefix_tokens} tokens")
        _check_prefill(wl, 0, f"prefill_f32_{seed}")


@pytest.mark.parametrize("g", [1, 2, 4, 8])
def test_prefill_attention_bf16_all_kernels(g):
    """Generic kernel and all shapes of the streaming kernel: segments shorter than a row
    block, segments of many row groups, empty headers, ragged ends."""
    wl = W.random_workload(92 + g, dtype="bf16", hq=8, hkv=8 // g, d=128, base=500000.0, t=2, p=3,
                           j_range=(1, 3), h_range=(0, 90), l_range=(1, 260 if g > 1 else 700))
    for mode in (0, 1, 3, 4):  # 0: the prefill's own kernel
        _say(f"prefill bf16 G={g} mode {mode}: {wl.n_prefix_tokens} tokens")
        rel = _check_prefill(wl, mode, f"prefill_bf16_g{g}_m{mode}")
        _say(f"  worst err/rms {rel:.2e}")


@pytest.mark.parametrize("literal", [False, True])
@pytest.mark.parametrize("g", [1, 3, 4, 8])
def test_prefill_attention_at_the_edges_of_its_blocks(g, literal):
    """The prefill kernel's rounds of two 32-key blocks: no header, headers that end inside or at
    the end of either block of a round, documents of one token, of a row group and one token more or
    less, an odd and an even number of blocks; 3 query heads per kv head run with a padding row."""
    grp = 128 // (4 if g == 3 else g)  # tokens per row group
    header = [0, 1, 31, 32, 33, 64, 95]
    per = [2, 1, 3, 2, 2, 1, 2]
    doc = [1, grp, grp + 1, 31, 33, 2 * grp - 1, 32, 64, 65, 3 * grp + 5, 96, 1, 97]
    n_doc = len(doc)
    attr = np.arange(n_doc).astype(np.int32) * 11 % 40 + 1 if literal else None
    from paper_2604_26209_amd import binding as B
    for hkv in (1, 2):
        wl = W.make_workload("edges", "bf16", g * hkv, hkv, 128, 500000.0, 2, header, per, doc, [1] * n_doc, [2] * n_doc)
        _say(f"prefill edges G={g} hkv={hkv} literal={literal}: {wl.n_prefix_tokens} tokens")
        rel = _check_prefill(wl, 0, f"prefill_edges_g{g}_{literal}", attr_len=attr)
        _say(f"  worst err/rms {rel:.2e}")
        # bf16 outputs are the fp32 outputs rounded to nearest even, nothing else
        outs = []
        for out_dtype, dt in ((B.HPD_OUT_F32, torch.float32), (B.HPD_OUT_SAME, torch.bfloat16)):
            layout = B.layout_from_workload(wl, out_dtype=out_dtype,
                                            **(dict(pos_mode=B.HPD_POS_PAPER_GAP, attr_len=attr,
                                                    mask_mode=B.HPD_MASK_PAPER) if literal else {}))
            n_tok = int(layout.counts()[B.HPD_C_N_PREFIX_TOKENS])
            inputs = H.Inputs(wl, layout.n_live(), "cuda", n_tok)
            q = W.normal_values((n_tok, g * hkv, 128), 5, "cuda", "bf16")
            kp, vp, _, _ = B.alloc_pools(layout)
            B.hpd_prefix_fill(layout, inputs.k_raw, inputs.v_raw, kp, vp)
            outs.append(torch.zeros((n_tok, g * hkv, 128), dtype=dt, device="cuda"))
            B.hpd_prefill_attention(layout, q, kp, vp, outs[-1])
        assert torch.equal(outs[0].to(torch.bfloat16), outs[1])


@pytest.mark.parametrize("literal", [False, True])
@pytest.mark.parametrize("g,hkv", [(1, 16), (2, 5), (3, 6), (4, 8), (8, 3)])
def test_prefill_attention_with_three_workgroups_per_cu(g, hkv, literal):
    """The same edges in a launch of more than two row groups per CU, which runs rounds of one block; a number of kv heads
    that is no multiple of 8 deals the row groups to several lanes."""
    grp = 128 // (4 if g == 3 else g)
    header, doc = [0, 1, 31, 32, 33, 64, 95], [1, grp, grp + 1, 31, 33, 2 * grp - 1, 32, 64, 65, 3 * grp + 5, 96, 1, 97]
    per = [2, 1, 3, 2, 2, 1, 2]
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    once = sum(-(-n // grp) for n in header + doc) * hkv
    n = 2 * cus // once + 1
    n_doc = len(doc) * n
    attr = np.arange(n_doc).astype(np.int32) * 11 % 40 + 1 if literal else None
    wl = W.make_workload("three", "bf16", g * hkv, hkv, 128, 500000.0, 2, header * n, per * n, doc * n, [1] * n_doc, [2] * n_doc)
    _say(f"prefill three per CU G={g} hkv={hkv} literal={literal}: {wl.n_prefix_tokens} tokens, {once * n} row groups")
    for change in (None, lambda q, k: (q * 8, k)):  # (and rows that a few keys dominate: the reference point moves often)
        rel = _check_prefill(wl, 0, f"prefill_three_g{g}_{literal}", attr_len=attr, change=change)
        _say(f"  worst err/rms {rel:.2e}")


@pytest.mark.parametrize("hkv", [1, 2])
def test_prefill_attention_of_a_list_of_row_groups_that_is_uploaded_by_itself(hkv):
    """More than 8192 row groups of 16 tokens per kv head, in several lanes: against the general kernel, which has no list."""
    from paper_2604_26209_amd import binding as B
    per, n = 12, 90
    doc = [113 + i % 16 for i in range(per * n)]
    wl = W.make_workload("long_list", "bf16", 8 * hkv, hkv, 128, 500000.0, 2, [33] * n, [per] * n, doc, [1] * len(doc), [2] * len(doc))
    q = W.normal_values((wl.n_prefix_tokens, 8 * hkv, 128), 5, "cuda", "bf16")
    k, v = (W.normal_values((wl.n_prefix_tokens, hkv, 128), seed, "cuda", "bf16") for seed in (6, 7))
    _say(f"prefill, long list, hkv={hkv}: {wl.n_prefix_tokens} tokens")
    outs = []
    for mode in (0, 3):
        lay = B.layout_from_workload(wl, out_dtype=B.HPD_OUT_F32)
        B.hpd_set_kernel_mode(lay, mode)
        kp, vp, _, _ = B.alloc_pools(lay)
        B.hpd_prefix_fill(lay, k, v, kp, vp)
        outs.append(torch.zeros(q.shape, device="cuda"))
        B.hpd_prefill_attention(lay, q, kp, vp, outs[-1])
    # two roundings of queries and weights to 11 bits, of outputs of size 1
    assert float((outs[0] - outs[1]).abs().max()) < H.BF16_TOL * float(outs[1].square().mean().sqrt())


@pytest.mark.parametrize("literal", [False, True])
@pytest.mark.parametrize("case", ["low", "very_low", "rising", "falling", "common_offset", "peaked_x8"])
def test_prefill_score_ranges_of_the_online_softmax(case, literal):
    """Prefill scores other than those of N(0,1).  Every score of a row near -150 or near -1000 in log2
    units; plateaus of 40 keys that rise from -1000 to +300, or fall; every score near +16; rows that one
    key or a few dominate.  Rows that start with one key (no header, the first header token) and rows behind a
    header.  The offsets are in channel 63, whose rotation is small at these positions: the rounding of
    the query there moves all keys of a plateau alike, so the tolerance stays the one of N(0,1) inputs.
    The prefill's own kernel and the general kernel."""
    wl = W.make_workload("scores", "bf16", 8, 2, 128, 500000.0, 2, [0, 1, 40, 129], [2, 2, 3, 1],
                         [1, 200, 33, 97, 64, 5, 150, 31], [1] * 8, [2] * 8)
    attr = np.arange(8).astype(np.int32) * 7 % 20 + 1 if literal else None

    def change(q, k):
        q, k = q.float(), k.float()
        if case == "peaked_x8":
            q = q * 8
        elif case == "common_offset":
            q, k = q + 1, k + 1
        else:
            a = 32.0 if case == "low" else 64.0
            level = dict(low=[-37.0], very_low=[-122.0], rising=[-122.0, -61.0, -30.0, 0.0, 16.0, 37.0],
                         falling=[37.0, 16.0, 0.0, -30.0, -61.0, -122.0])[case]
            at = torch.arange(k.shape[0], device=k.device) // 40 % len(level)
            q[..., 63] = a
            k[..., 63] = torch.tensor(level, device=k.device)[at][:, None]
        return q.to(torch.bfloat16), k.to(torch.bfloat16)

    for mode in (0, 4):
        _say(f"prefill score ranges: {case} literal={literal} mode {mode}")
        rel = _check_prefill(wl, mode, f"prefill_{case}_{literal}_m{mode}", attr_len=attr, change=change)
        _say(f"  worst err/rms {rel:.2e}")


def test_prefill_scores_far_above_the_first_reference_point():
    """192 keys with scores near -8356 in log2 units, then keys with scores near 0, which decide: their weights
    must not carry the rounding of the first ones' scores (up to 5e-4 in every sum around 8000).  Error against
    the oracle in 64 bits over the rows that see both, relative 2-norm; the general kernel, which adds every
    score up from 0, is the measure.  10 %: right after the jump the largest weight of a row is 1 to within that
    rounding instead of exactly, and is rounded to half as the others are.  (With the rounding: 2.4 times.)"""
    from paper_2604_26209_amd import binding as B
    n = 1000
    wl = W.make_workload("jump", "bf16", 8, 2, 128, 500000.0, 2, [0], [1], [n], [1], [2])
    err = {}
    for mode in (0, 4):
        layout = B.layout_from_workload(wl, out_dtype=B.HPD_OUT_F32)
        B.hpd_set_kernel_mode(layout, mode)
        inp = H.Inputs(wl, layout.n_live(), "cuda")
        q = W.normal_values((n, 8, 128), 5, "cuda", "bf16")
        q[..., 63] = 64.0
        inp.k_raw[..., 63] = (torch.arange(n, device="cuda") < 192)[:, None] * -1024.0
        kp, vp, _, _ = B.alloc_pools(layout)
        B.hpd_prefix_fill(layout, inp.k_raw, inp.v_raw, kp, vp)
        out = torch.full((n, 8, 128), float("nan"), device="cuda")
        B.hpd_prefill_attention(layout, q, kp, vp, out)
        orc = O.HPDOracle(wl.header_len, wl.doc_ptr, wl.doc_len, wl.branch_ptr, wl.branch_len, 8, 2, 128, 500000.0, 2,
                          dtype=np.float64, cache_dtype="bf16")
        orc.prefill({0: inp.k_raw.double().cpu().numpy()}, {0: inp.v_raw.double().cpu().numpy()})
        want = orc.prefill_attention({0: q.double().cpu().numpy()})[0][192:]
        got = out.double().cpu().numpy()[192:]
        err[mode] = float(np.linalg.norm(got - want) / np.linalg.norm(want))
    _say(f"prefill scores above the reference point: {err[0]:.3e}, general kernel {err[4]:.3e}")
    assert err[0] <= 1.1 * err[4]


def _error(got, want):
    return float(np.linalg.norm(got.double().cpu().numpy() - want) / np.linalg.norm(want))


def test_prefill_error_with_three_workgroups_per_cu_is_no_larger():
    """One prompt by itself (two workgroups per CU, rounds of two blocks) and as the first of sixteen (three, of one block): error
    of its rows against the oracle in 64 bits.  With a reference point from the first block alone it was 0.8 % larger; 0.2 % is
    what the order of the sums may add."""
    from paper_2604_26209_amd import binding as B
    err = {}
    for n in (16, 1):
        wl = W.make_workload("error", "bf16", 32, 8, 128, 500000.0, 2, [64] * n, [1] * n, [512] * n, [1] * n, [2] * n)
        layout = B.layout_from_workload(wl, out_dtype=B.HPD_OUT_F32)
        if n == 16:
            inp = H.Inputs(wl, layout.n_live(), "cuda")
            q = W.normal_values((wl.n_prefix_tokens, 32, 128), 5, "cuda", "bf16")
        k, v, q = (x[:wl.n_prefix_tokens].contiguous() for x in (inp.k_raw, inp.v_raw, q))
        kp, vp, _, _ = B.alloc_pools(layout)
        B.hpd_prefix_fill(layout, k, v, kp, vp)
        out = torch.zeros(q.shape, device="cuda")
        B.hpd_prefill_attention(layout, q, kp, vp, out)
        err[n] = out[:576]
    orc = O.HPDOracle(wl.header_len, wl.doc_ptr, wl.doc_len, wl.branch_ptr, wl.branch_len, 32, 8, 128, 500000.0, 2,
                      dtype=np.float64, cache_dtype="bf16")
    orc.prefill({0: k.double().cpu().numpy()}, {0: v.double().cpu().numpy()})
    want = orc.prefill_attention({0: q.double().cpu().numpy()})[0]
    err = {n: _error(x, want) for n, x in err.items()}
    _say(f"prefill error: two workgroups per CU {err[1]:.4e}, three {err[16]:.4e}")
    assert err[16] <= 1.002 * err[1]


def test_decode_error_with_three_workgroups_per_cu_is_no_larger():
    """The same of a literal decode step with many rows per unit: the first 8 prompts of 24 (384 workgroups) and of 48 (768).  It was
    1 % larger."""
    from paper_2604_26209_amd import binding as B
    outs, kw = {}, {}
    for n in (48, 24):
        wl = W.make_workload("error", "bf16", 64, 8, 128, 500000.0, 1, [64] * n, [2] * n, [72] * (2 * n), [16] * (2 * n), [1] * (32 * n))
        kw = dict(pos_mode=B.HPD_POS_PAPER_GAP, attr_len=np.ones(32 * n, np.int32), mask_mode=B.HPD_MASK_PAPER)
        if n == 48:
            a = H.run_hip(wl, fused=True, **kw)
            inp = a["inputs"]
        else:
            lay = B.layout_from_workload(wl, **kw)
            tok, live = int(lay.counts()[B.HPD_C_N_PREFIX_TOKENS]), int(lay.n_live()[0])
            inp.k_raw, inp.v_raw = inp.k_raw[:tok].contiguous(), inp.v_raw[:tok].contiguous()
            inp.q, inp.k_new, inp.v_new = ([x[0][:live].contiguous()] for x in (inp.q, inp.k_new, inp.v_new))
            a = H.run_hip(wl, inputs=inp, fused=True, **kw)
        outs[n] = a["out"][0]
    _, res = H.run_oracle(wl, inp, prompts=list(range(8)), pos_mode="paper_gap", attr_len=kw["attr_len"], mask_mode="paper")
    rows = torch.from_numpy(res[0]["rows"]).cuda()
    err = {n: _error(x[rows], res[0]["out"].astype(np.float64)) for n, x in outs.items()}
    _say(f"literal decode error: two workgroups per CU {err[24]:.4e}, three {err[48]:.4e}")
    assert err[48] <= 1.002 * err[24]


def test_prefill_attention_literal_mask_fp32_generic():
    """First inference step under HPD_MASK_PAPER: header, stacked documents and attribute names
    as one causal sequence; the names' rows are the ones whose outputs start the branches."""
    for seed, kw in [(95, dict(hq=4, hkv=2, d=64, t=3, p=3, j_range=(1, 3), h_range=(0, 20), l_range=(1, 70))),
                     (96, dict(hq=2, hkv=2, d=32, t=2, p=2, h_range=(0, 0), l_range=(1, 5)))]:
        wl = W.random_workload(seed, dtype="f32", **kw)
        attr = np.random.default_rng(seed).integers(1, 5, size=wl.n_branches).astype(np.int32)
        _say(f"prefill literal f32 seed {seed}: {wl.n_prefix_tokens} + {int(attr.sum())} tokens")
        _check_prefill(wl, 0, f"prefill_literal_f32_{seed}", attr_len=attr)


@pytest.mark.parametrize("g", [1, 2, 4, 8])
def test_prefill_attention_literal_mask_bf16_all_kernels(g):
    wl = W.random_workload(97 + g, dtype="bf16", hq=8, hkv=8 // g, d=128, base=500000.0, t=2, p=3,
                           j_range=(1, 4), n_range=(1, 30), h_range=(0, 90), l_range=(1, 200 if g > 1 else 500))
    attr = np.random.default_rng(97 + g).integers(1, 5, size=wl.n_branches).astype(np.int32)
    for mode in (0, 1, 3, 4):
        _say(f"prefill literal bf16 G={g} mode {mode}: {wl.n_prefix_tokens} + {int(attr.sum())} tokens")
        rel = _check_prefill(wl, mode, f"prefill_literal_bf16_g{g}_m{mode}", attr_len=attr)
        _say(f"  worst err/rms {rel:.2e}")


@pytest.mark.parametrize("literal", [False, True])
def test_prefix_fill_fast_kernel_equals_general_kernel(literal):
    """hpd_prefix_fill for bf16 / 128 channels (16-byte moves, V interleave through LDS, V padding
    zeroed in the same pass) against the element-wise kernel (kernel_mode 1): the same bits in
    every slot of both pools, ragged segments, empty headers, attribute-name segments."""
    from paper_2604_26209_amd import binding as B
    wl = W.random_workload(170 + int(literal), dtype="bf16", hq=8, hkv=2, d=128, base=500000.0, t=3, p=4,
                           j_range=(1, 4), n_range=(1, 12), h_range=(0, 70), l_range=(1, 150))
    attr = np.random.default_rng(170).integers(1, 5, size=wl.n_branches).astype(np.int32)
    kw = dict(pos_mode=B.HPD_POS_PAPER_GAP, attr_len=attr, mask_mode=B.HPD_MASK_PAPER) if literal else {}
    pools = []
    for mode in (0, 1):
        lay = B.layout_from_workload(wl, **kw)
        if mode:
            B.hpd_set_kernel_mode(lay, mode)
        n_tok = int(lay.counts()[B.HPD_C_N_PREFIX_TOKENS])
        k_raw = W.normal_values((n_tok, wl.n_kv_heads, wl.head_dim), 1, "cuda", wl.dtype)
        v_raw = W.normal_values((n_tok, wl.n_kv_heads, wl.head_dim), 2, "cuda", wl.dtype)
        kp, vp, _, _ = B.alloc_pools(lay)
        kp.fill_(3.0), vp.fill_(3.0)  # K padding is left alone by both kernels
        B.hpd_prefix_fill(lay, k_raw, v_raw, kp, vp)
        pools.append((kp, vp))
    torch.cuda.synchronize()
    _say(f"prefix fill, literal {literal}: {n_tok} tokens, {pools[0][0].numel()} pool elements")
    assert torch.equal(pools[0][0].view(torch.int16), pools[1][0].view(torch.int16))
    assert torch.equal(pools[0][1].view(torch.int16), pools[1][1].view(torch.int16))
    assert bool((pools[0][0] != 3.0).any())


@pytest.mark.parametrize("hkv,docs", [(4, 300), (12, 100), (6, 200), (16, 40)])
def test_prefix_fill_of_large_batches_equals_general_kernel(hkv, docs):
    """Launches of 16384 (block, kv head) and more, four heads a workgroup where the heads divide by four (6 do not, and 16
    x 40 documents stay below): the bits of the element-wise kernel, infinities included, in ragged segments."""
    from paper_2604_26209_amd import binding as B
    doc = [1 + 977 * i % 1500 for i in range(docs)]
    wl = W.make_workload("fill", "bf16", hkv, hkv, 128, 500000.0, 2, [0, 45], [docs // 2, docs - docs // 2], doc, [1] * docs, [2] * docs)
    pools = []
    for mode in (0, 1):
        lay = B.layout_from_workload(wl)
        B.hpd_set_kernel_mode(lay, mode)
        k_raw, v_raw = (W.normal_values((wl.n_prefix_tokens, hkv, 128), i, "cuda", "bf16") for i in (1, 2))
        k_raw[3, 1, 5], v_raw[7, 0, 70], v_raw[8, 1, 3] = float("inf"), float("-inf"), 1e-30
        kp, vp, _, _ = B.alloc_pools(lay)
        kp.fill_(3.0), vp.fill_(3.0)
        B.hpd_prefix_fill(lay, k_raw, v_raw, kp, vp)
        pools.append((kp.view(torch.int16), vp.view(torch.int16)))
    _say(f"prefix fill, {wl.n_prefix_tokens} tokens x {hkv} heads: {pools[0][0].numel() // (32 * 128)} (block, kv head)")
    assert torch.equal(pools[0][0], pools[1][0]) and torch.equal(pools[0][1], pools[1][1])


def _finetune_mask_of_all_pairs(plen, al, vl):
    """The rule over codes (attribute, k) of all pairs, as in the docstring of the oracle's loop."""
    owner = np.concatenate([np.full(plen, -1)] + [np.full(a + v, n) for n, (a, v) in enumerate(zip(al, vl))])
    k = np.concatenate([np.zeros(plen, int)] + [np.r_[np.zeros(a, int), 1:v + 1] for a, v in zip(al, vl)])
    value, name = k > 0, (k == 0) & (owner >= 0)
    ok = np.tri(len(k), dtype=bool) & ~(value[None] & name[:, None])
    ok &= ~(value[None] & value[:, None] & (owner[None] < owner[:, None]) & (k[None] > k[:, None]))
    return ok.astype(np.uint8)


@pytest.mark.parametrize("n_attr", [0, 1, 640, 641])
@pytest.mark.parametrize("plen", [0, 15, 16, 4090])
def test_finetune_mask_at_the_edges_of_its_blocks(plen, n_attr):
    """Sequences that are no multiple of the 16 keys of a thread, of the 8 queries and 4096 keys of a workgroup,
    the number of attributes around what travels in the kernel's arguments, with and without positions."""
    from oracle import finetune_mask as F
    from paper_2604_26209_amd import binding as B
    al, vl = 1 + np.arange(n_attr) % 3, np.arange(n_attr) * 5 % 4
    if n_attr == 1:
        vl = np.array([37])
    kmax = 40
    s = plen + int(al.sum() + vl.sum())
    _say(f"finetune mask edges: prompt {plen}, {n_attr} attributes, {s} tokens")
    assert B.hpd_finetune_mask(plen, al, vl, kmax) == s
    if s == 0:
        return
    pos = torch.full((s + 8,), -7, dtype=torch.int32, device="cuda")
    m = torch.full((s * s + 64,), 9, dtype=torch.uint8, device="cuda")
    B.hpd_finetune_mask(plen, al, vl, kmax, pos[:s], m[:s * s].view(s, s))
    assert np.array_equal(pos[:s].cpu().numpy(), F.finetune_position_ids(plen, al, vl, kmax))
    assert bool((pos[s:] == -7).all()) and bool((m[s * s:] == 9).all())
    assert np.array_equal(m[:s * s].view(s, s).cpu().numpy(), _finetune_mask_of_all_pairs(plen, al, vl))


@pytest.mark.parametrize("s", [1, 15, 16, 17, 31, 388, 4097, 4111, 4112, 4113])
def test_finetune_mask_of_any_number_of_tokens(s):
    """Lengths around the 16 keys of a thread, alone and behind the 4096 keys of a workgroup, with a value at the end."""
    from paper_2604_26209_amd import binding as B
    al, vl = ([], []) if s < 3 else ([1, 1], [s // 3, 1]) if s < 17 else ([2, 1], [8, 5])
    plen = s - sum(al) - sum(vl)
    _say(f"finetune mask of {s} tokens")
    m = torch.full((s * s + 64,), 9, dtype=torch.uint8, device="cuda")
    B.hpd_finetune_mask(plen, al, vl, 40, None, m[:s * s].view(s, s))
    assert bool((m[s * s:] == 9).all())
    want = _finetune_mask_of_all_pairs(plen, np.array(al, int), np.array(vl, int))
    assert np.array_equal(m[:s * s].view(s, s).cpu().numpy(), want)


@pytest.mark.parametrize("s,off", [(16, 1), (17, 15), (1007, 3), (1008, 8), (1023, 12), (1024, 5), (1025, 0), (4031, 7), (4032, 1),
                                   (4033, 14), (4047, 2), (4048, 9), (8065, 11), (11600, 6)])
def test_finetune_mask_at_any_address(s, off):
    """A mask that starts anywhere, of lengths around the 63 x 16 keys of a wave and the 4032 of a workgroup: rows begin
    and end inside a 16-byte unit of the memory; the longest is written past the L2's write-through limit."""
    from paper_2604_26209_amd import binding as B
    n = s // 40
    al, vl = 1 + np.arange(n) % 3, np.arange(n) * 7 % 30
    plen = s - int(al.sum() + vl.sum())
    _say(f"finetune mask of {s} tokens at byte {off}")
    buf = torch.full((s * s + 64,), 9, dtype=torch.uint8, device="cuda")
    m = buf[off:off + s * s]
    assert B.hpd_finetune_mask(plen, al, vl, 40, None, m) == s
    assert bool((buf[:off] == 9).all()) and bool((buf[off + s * s:] == 9).all())
    owner = torch.full((s,), -1, dtype=torch.int32, device="cuda")
    k, at = torch.zeros_like(owner), plen
    for a, (x, y) in enumerate(zip(al.tolist(), vl.tolist())):
        owner[at:at + x + y] = a
        k[at + x:at + x + y] = torch.arange(1, y + 1, device="cuda")
        at += x + y
    i = torch.arange(s, device="cuda")
    ok = i[None] <= i[:, None]
    ok &= ~((k[None] > 0) & ((k == 0) & (owner >= 0))[:, None])
    ok &= ~((k[None] > k[:, None]) & (k[:, None] > 0) & (owner[None] < owner[:, None]))
    assert torch.equal(m.view(s, s), ok.to(torch.uint8))


@pytest.mark.parametrize("n_attr", [7, 650])
def test_finetune_mask_of_long_values(n_attr):
    """Values around and far above the 64 tokens that one thread expands, across the 4096 keys of a workgroup; with a
    mask only, with positions only, with the offsets in the kernel's arguments and in memory."""
    from oracle import finetune_mask as F
    from paper_2604_26209_amd import binding as B
    al, vl = np.ones(n_attr, int), np.zeros(n_attr, int)
    vl[:7] = [65, 64, 3900, 0, 300, 66, 1]
    vl[-1] = 70
    plen, kmax = 5, 4000
    s = plen + int(al.sum() + vl.sum())
    _say(f"finetune mask of long values: {n_attr} attributes, {s} tokens")
    m = torch.full((s, s), 9, dtype=torch.uint8, device="cuda")
    pos = torch.full((s,), -7, dtype=torch.int32, device="cuda")
    B.hpd_finetune_mask(plen, al, vl, kmax, None, m)
    B.hpd_finetune_mask(plen, al, vl, kmax, pos, None)
    assert np.array_equal(pos.cpu().numpy(), F.finetune_position_ids(plen, al, vl, kmax))
    assert np.array_equal(m.cpu().numpy(), _finetune_mask_of_all_pairs(plen, al, vl))


def test_finetune_mask_of_one_long_value_takes_no_longer():
    """The mask of 4004 tokens, all but a hundred of one value, against the same number of tokens in 128 attributes: the
    bytes written are the same.  (One thread for the value: 6.7 times; 2 leaves room for two timings.)"""
    from paper_2604_26209_amd import binding as B
    m = torch.zeros(4004, 4004, dtype=torch.uint8, device="cuda")
    us = []
    for plen, al, vl, kmax in ((100, [4], [3900], 4000), (2596, [3] * 128, [8] * 128, 16)):
        best = 1e9
        for _ in range(20):
            start, end = torch.cuda.Event(True), torch.cuda.Event(True)
            start.record()
            for _ in range(5):
                B.hpd_finetune_mask(plen, al, vl, kmax, None, m)
            end.record()
            torch.cuda.synchronize()
            best = min(best, start.elapsed_time(end) * 200)
        us.append(best)
    _say(f"finetune mask: one value of 3900 tokens {us[0]:.1f} us, 128 attributes {us[1]:.1f} us")
    assert us[0] <= 2 * us[1]


def test_finetune_mask_and_positions_bit_exact():
    """hpd_finetune_mask (Section 4.4) against the loop oracle: mask and position IDs."""
    from oracle import finetune_mask as F
    from paper_2604_26209_amd import binding as B
    rng = np.random.default_rng(9)
    cases = [(10, [3, 3, 3], [3, 3, 3], 7), (0, [1], [1], 1), (4, [2, 1, 3], [0, 5, 2], 5)]
    for _ in range(4):
        n = int(rng.integers(1, 20))
        kmax = int(rng.integers(1, 31))
        cases.append((int(rng.integers(0, 100)), [int(x) for x in rng.integers(1, 6, n)],
                      [int(x) for x in rng.integers(0, kmax + 1, n)], kmax))
    for plen, al, vl, kmax in cases:
        _say(f"finetune mask: prompt {plen}, {len(al)} attributes, K_max {kmax}")
        s = B.hpd_finetune_mask(plen, al, vl, kmax)
        assert s == plen + sum(al) + sum(vl)
        pos = torch.full((s,), -7, dtype=torch.int32, device="cuda")
        m = torch.full((s, s), 7, dtype=torch.uint8, device="cuda")
        B.hpd_finetune_mask(plen, al, vl, kmax, pos, m)
        assert np.array_equal(pos.cpu().numpy(), F.finetune_position_ids(plen, al, vl, kmax))
        assert np.array_equal(m.cpu().numpy(), F.finetune_mask(plen, al, vl))


def test_mask_export_bit_exact():
    from paper_2604_26209_amd import binding as B
    _say("mask export")
    wl = W.random_workload(31, dtype="f32", t=4, p=3, l_range=(1, 30), h_range=(0, 12))
    hip = H.run_hip(wl)
    orc, _ = H.run_oracle(wl, hip["inputs"])
    for p, po in orc.prompts.items():
        s = B.hpd_expand_mask(hip["layout"], p, wl.max_new - 1)
        assert s == len(po.kind)
        m = torch.full((s, s), 7, dtype=torch.uint8, device="cuda")
        B.hpd_expand_mask(hip["layout"], p, wl.max_new - 1, m)
        assert np.array_equal(m.cpu().numpy(), po.dense_mask())


@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("g", [1, 3, 5, 16])
def test_fp32_decode_kernel_at_the_edges_of_its_tiles(g, d):
    """Row groups of 16 rows (16, 5, 3 and 1 branches), tiles of 16 keys: headers and documents around a
    tile, no header, one branch, exactly one row group and one branch more, branches that end (so
    that a document's live branches are no run of ids), tails of 1 to 12 positions.  Against the
    oracle, the step call against the two-call sequence, and against the generic kernel (fp32 sums of
    at most 200 terms of size 1 in another order: 1e-5)."""
    hkv, per_group = 2, 16 // g
    header, per, doc = [0, 1, 16, 33], [2, 1, 2, 1], [1, 15, 17, 160, 32, 47]
    nbr = [1, per_group, per_group + 1, 2, 2 * per_group + 1, 3]
    blen = 1 + np.arange(sum(nbr)) * 7 % 12
    wl = W.make_workload("f32edges", "f32", g * hkv, hkv, d, 10000.0, 12, header, per, doc, nbr, blen)
    _say(f"fp32 decode edges G={g} D={d}")
    two = H.run_hip(wl)
    worst = H.check_all(wl, two, label=f"f32_edges_g{g}_d{d}")
    one = H.run_hip(wl, inputs=two["inputs"], fused=True)
    gen = H.run_hip(wl, inputs=two["inputs"], kernel_mode=1)
    for x, y, z in zip(two["out"], one["out"], gen["out"]):
        assert torch.equal(x, y)
        assert x.numel() == 0 or float((x - z).abs().max()) < 1e-5
    # it was the kernel of its own that ran: sums in another order are not the same bits throughout
    assert not all(torch.equal(x, z) for x, z in zip(two["out"], gen["out"]))
    _say(f"  max-abs against the oracle {worst:.2e}")


def test_fp32_decode_with_pools_off_16_bytes_runs_the_generic_kernel():
    """The fp32 kernel loads 16 bytes at a time; pools that start 4 bytes off give the generic kernel's bits."""
    from paper_2604_26209_amd import binding as B
    wl = W.make_workload("off16", "f32", 8, 2, 64, 10000.0, 3, [20], [2], [50, 7], [5, 3], [3] * 8)
    outs = {}
    for mode, off in ((0, 0), (0, 1), (1, 0)):
        layout = B.layout_from_workload(wl)
        B.hpd_set_kernel_mode(layout, mode)
        inputs = H.Inputs(wl, layout.n_live(), "cuda")
        pools = []
        for x in B.alloc_pools(layout):
            pools.append(torch.zeros(x.numel() + 4, device="cuda")[off:off + x.numel()])
        kp, vp, kt, vt = pools
        B.hpd_prefix_fill(layout, inputs.k_raw, inputs.v_raw, kp, vp)
        outs[mode, off] = []
        for t in range(3):
            out = torch.zeros_like(inputs.q[t])
            B.hpd_decode_step(layout, t, inputs.q[t], inputs.k_new[t], inputs.v_new[t], kp, vp, kt, vt, out)
            outs[mode, off].append(out)
    same = [all(torch.equal(x, y) for x, y in zip(outs[0, off], outs[1, 0])) for off in (0, 1)]
    assert same == [False, True]


@pytest.mark.parametrize("d", [32, 64, 128])
def test_fp32_decode_with_tail_values_off_16_bytes_and_long_tails(d):
    """Tail values that start 4 bytes off are fetched a float at a time: the bits of the aligned pool.  40 steps, so that
    a tile holds the ends of branches of 1, 15, 16, 17 and more tokens; against the generic kernel (fp32 sums of at most 80
    terms of size 1 in another order: 1e-5)."""
    from paper_2604_26209_amd import binding as B
    wl = W.make_workload("vtail4", "f32", 4, 2, d, 10000.0, 40, [3], [3], [40, 7, 1], [1, 5, 9], [40, 40, 1, 17, 40, 33] + [40] * 9)
    _say(f"fp32 decode, tail values off 16 bytes, D={d}")
    outs = {}
    for mode, off in ((0, 0), (0, 1), (1, 0)):
        layout = B.layout_from_workload(wl)
        B.hpd_set_kernel_mode(layout, mode)
        inputs = H.Inputs(wl, layout.n_live(), "cuda")
        kp, vp, kt, vt = B.alloc_pools(layout)
        vt = torch.full((vt.numel() + 4,), float("nan"), device="cuda")[off:off + vt.numel()]
        B.hpd_prefix_fill(layout, inputs.k_raw, inputs.v_raw, kp, vp)
        outs[mode, off] = []
        for t in range(wl.max_new):
            out = torch.zeros_like(inputs.q[t])
            B.hpd_decode_step(layout, t, inputs.q[t], inputs.k_new[t], inputs.v_new[t], kp, vp, kt, vt, out)
            outs[mode, off].append(out)
    for x, y, z in zip(outs[0, 0], outs[0, 1], outs[1, 0]):
        assert torch.equal(x, y)
        assert float((x - z).abs().max()) < 1e-5


@pytest.mark.parametrize("d,page", [(64, 0), (128, 8)])
def test_fp32_decode_with_tail_values_off_16_bytes_takes_little_longer(d, page):
    """Long tails: the rows of a tile are looked up once, also where its values are fetched a float at a time.  (Looked up
    for every such instruction, these steps took 2.0 and 4.2 times the time of aligned values.)"""
    from paper_2604_26209_amd import binding as B
    steps, n = 128, 12
    wl = W.make_workload("vtail4", "f32", 16, 4, d, 10000.0, steps, [0] * 64, [1] * 64, [20] * 64, [n] * 64, [steps] * (64 * n))
    lay = B.layout_from_workload(wl)
    if page:
        pages = wl.n_branches * steps // page
        table = torch.randperm(pages, device="cuda").to(torch.int32).view(wl.n_branches, -1).contiguous()
        B.hpd_set_tail_pages(lay, page, pages, table)
    kp, vp, kt, vt = (x.normal_() for x in B.alloc_pools(lay))
    off = torch.randn(vt.numel() + 4, device="cuda")[1:vt.numel() + 1]
    q, k, v = (torch.randn(wl.n_branches, h, d, device="cuda") for h in (16, 4, 4))
    out = torch.zeros_like(q)
    us = _us_in_turn([lambda x=x: B.hpd_decode_step(lay, 120, q, k, v, kp, vp, kt, x, out) for x in (vt, off)])
    _say(f"fp32 decode, D={d}, page {page}: {us[0]:.1f} us, tail values off 16 bytes {us[1]:.1f} us")
    assert us[1] < 1.6 * us[0]


def test_fp32_decode_of_two_units_uses_the_whole_chip():
    """The row groups of a (unit, kv head) run on one XCD to share its L2, but not where that leaves XCDs without work: two
    documents take less time than eight (on an XCD each, they took the same)."""
    from paper_2604_26209_amd import binding as B
    steps, n, calls = 64, 50, []
    for docs in (2, 8):
        wl = W.make_workload("xcds", "f32", 16, 1, 64, 10000.0, steps, [100] * docs, [1] * docs, [600] * docs, [n] * docs, [steps] * (docs * n))
        lay = B.layout_from_workload(wl)
        pools = [x.normal_() for x in B.alloc_pools(lay)]
        q, k, v = (torch.randn(wl.n_branches, h, 64, device="cuda") for h in (16, 1, 1))
        out = torch.zeros_like(q)
        calls.append(lambda lay=lay, q=q, k=k, v=v, pools=pools, out=out: B.hpd_decode_step(lay, 55, q, k, v, *pools, out))
    us = _us_in_turn(calls)
    _say(f"fp32 decode, two units {us[0]:.1f} us, eight {us[1]:.1f} us")
    assert us[0] < 0.85 * us[1]


# fp32 batches whose rows fill the 16-row groups badly: heads, channels, documents, branches of each
# document, steps
F32_UNEVEN = {
    "one_document_of_many_branches": (16, 4, 64, [40] * 10 + [64], [1] * 5 + [0] + [2] * 4 + [41], 5),
    "one_long_document": (8, 8, 32, [3] * 299 + [400], [1] * 300, 3),
    "tails_longer_than_the_document": (6, 2, 32, [17, 3], [11, 16], 40),
    "one_row_per_document": (8, 8, 128, [5] * 100, [1] * 100, 1),
    "short_documents_of_many_heads": (16, 1, 128, [3], [2], 2),
}

F32_GENERIC = ("one_row_per_document", "short_documents_of_many_heads")


@pytest.mark.parametrize("case", F32_UNEVEN)
def test_fp32_decode_of_uneven_batches(case):
    """The ways in which an fp32 step is cut into workgroups: against the oracle, the step call against the two-call
    sequence, and against the generic kernel (sums of at most 500 terms of size 1 in another order: 1e-5), whose
    bits tell which of the two kernels the layout's plan chose."""
    hq, hkv, d, doc, nbr, steps = F32_UNEVEN[case]
    blen = 1 + np.arange(sum(nbr)) * 3 % steps
    blen[-1] = steps
    wl = W.make_workload("uneven", "f32", hq, hkv, d, 10000.0, steps, [20, 0], [len(doc) // 2, len(doc) - len(doc) // 2],
                         doc, nbr, blen)
    _say(f"fp32 decode, {case}")
    two = H.run_hip(wl)
    worst = H.check_all(wl, two, label=case)
    one = H.run_hip(wl, inputs=two["inputs"], fused=True)
    gen = H.run_hip(wl, inputs=two["inputs"], kernel_mode=1)
    for x, y, z in zip(two["out"], one["out"], gen["out"]):
        assert torch.equal(x, y)
        assert x.numel() == 0 or float((x - z).abs().max()) < 1e-5
    assert all(torch.equal(x, z) for x, z in zip(two["out"], gen["out"])) == (case in F32_GENERIC)
    _say(f"  max-abs against the oracle {worst:.2e}")


F32_UNEVEN_LARGE = {
    "one_document_of_many_branches": (16, 4, 64, [64] * 1001, [1] * 1000 + [1000], 2),
    "one_long_document": (8, 8, 32, [3000] + [20] * 3000, [3] * 3001, 2),
    "tails_longer_than_the_document": (4, 4, 64, [32], [16], 401),
    "one_row_per_document": (8, 8, 128, [20] * 1000, [1] * 1000, 1),
}


@pytest.mark.parametrize("case", F32_UNEVEN_LARGE)
def test_fp32_decode_of_uneven_batches_is_no_slower_than_the_generic_kernel(case):
    """Where the default of an fp32 step cuts a batch badly it costs many times what the generic kernels take; 1.25 is
    well above what two timings of the same call differ by."""
    from paper_2604_26209_amd import binding as B
    hq, hkv, d, doc, nbr, steps = F32_UNEVEN_LARGE[case]
    wl = W.make_workload("uneven", "f32", hq, hkv, d, 10000.0, steps, [0], [len(doc)], doc, nbr, [steps] * sum(nbr))
    layout = B.layout_from_workload(wl)
    pools = B.alloc_pools(layout)
    for x in pools:
        x.normal_()
    n = wl.n_branches
    q, k, v = (torch.randn(n, h, d, device="cuda") for h in (hq, hkv, hkv))
    out = torch.zeros_like(q)
    us = {}
    for mode in (0, 1, 0, 1):
        B.hpd_set_kernel_mode(layout, mode)
        call = lambda: B.hpd_decode_step(layout, steps - 1, q, k, v, *pools, out)
        call()
        start, end = torch.cuda.Event(True), torch.cuda.Event(True)
        for _ in range(5):
            start.record()
            for _ in range(10):
                call()
            end.record()
            torch.cuda.synchronize()
            us[mode] = min(us.get(mode, 1e9), start.elapsed_time(end) * 100)
    _say(f"fp32 decode, {case}: {us[0]:.1f} us, generic kernels {us[1]:.1f} us")
    assert us[0] <= 1.25 * us[1]


@pytest.mark.parametrize("dtype,mode", [("f32", 0), ("f32", 1), ("bf16", 1)])
def test_a_refused_decode_step_leaves_the_tails_alone(dtype, mode):
    """A step whose rows see more keys than the generic kernel's LDS holds is refused before its append."""
    from paper_2604_26209_amd import binding as B
    d = 128 if dtype == "bf16" else 32
    wl = W.make_workload("too_long", dtype, 2, 1, d, 10000.0, 2, [0], [1], [15000], [3], [2] * 3)
    layout = B.layout_from_workload(wl)
    B.hpd_set_kernel_mode(layout, mode)
    kp, vp, kt, vt = B.alloc_pools(layout)
    for x in (kp, vp, kt, vt):
        x.fill_(3.0)
    inputs = H.Inputs(wl, layout.n_live(), "cuda")
    out = torch.full_like(inputs.q[0], 3.0)
    with pytest.raises(B.HpdError):
        B.hpd_decode_step(layout, 0, inputs.q[0], inputs.k_new[0], inputs.v_new[0], kp, vp, kt, vt, out)
    for x in (kt, vt, out):
        assert bool((x == 3.0).all())


def test_fp32_decode_kernel_keeps_infinite_values_in_their_branch():
    """A branch whose newest value is infinite or NaN: the other branches' rows, which share its tile, stay as
    they are without it."""
    from paper_2604_26209_amd import binding as B
    wl = W.make_workload("f32inf", "f32", 4, 2, 64, 10000.0, 4, [5], [1], [40], [11], [4] * 11)
    layout = B.layout_from_workload(wl)
    inputs = H.Inputs(wl, layout.n_live(), "cuda")
    outs = []
    for bad in (False, True):
        kp, vp, kt, vt = B.alloc_pools(layout)
        B.hpd_prefix_fill(layout, inputs.k_raw, inputs.v_raw, kp, vp)
        v = [x.clone() for x in inputs.v_new]
        if bad:
            v[1][3, 0, 7], v[2][9, 1, 8] = float("inf"), float("nan")
        for t in range(4):
            out = torch.zeros(11, 4, 64, device="cuda")
            B.hpd_decode_step(layout, t, inputs.q[t], inputs.k_new[t], v[t], kp, vp, kt, vt, out)
        outs.append(out.cpu())
    same = torch.ones(11, 4, 64, dtype=torch.bool)
    same[3, :2, 7], same[9, 2:, 8] = False, False
    assert torch.equal(outs[0][same], outs[1][same])
    assert not torch.isfinite(outs[1][~same]).any()


def test_kv_pools_hold_rotated_keys_at_reported_slots():
    """K tail and prefix pools against the oracle's cache (rotated K), through the
    documented pool layouts."""
    from paper_2604_26209_amd import binding as B
    _say("pool contents")
    wl = W.random_workload(51, dtype="f32", hq=4, hkv=2, d=64, t=4, p=2)
    hip = H.run_hip(wl, poison_pools="zero")
    orc, res = H.run_oracle(wl, hip["inputs"])
    kp, vp, kt, vt = [x.cpu().numpy() for x in hip["pools"]]
    lay = hip["layout"]
    c = lay.counts()
    NP, T, Hkv, D = int(c[B.HPD_C_N_PREFIX_SLOTS]), wl.max_new, wl.n_kv_heads, wl.head_dim
    kp = kp.reshape(Hkv, NP, D)
    vp = vp.reshape(Hkv, NP // 8, D, 8)
    kt = kt.reshape(wl.n_branches, Hkv, T, D)
    vt = vt.reshape(wl.n_branches, Hkv, T, D)
    seg_off = B.hpd_layout_query(lay, B.HPD_Q_SEG_OFF)
    for p, po in orc.prompts.items():
        segs = [(p, 0, po.h)]
        run = po.h
        for j, d in enumerate(range(wl.doc_ptr[p], wl.doc_ptr[p + 1])):
            segs.append((wl.n_prompts + d, run, po.doc_lens[j]))
            run += po.doc_lens[j]
        for sid, first, n in segs:
            for i in range(n):
                slot = seg_off[sid] + i
                assert np.abs(kp[:, slot, :] - po.k[first + i]).max() < 1e-5
                assert np.array_equal(vp[:, slot // 8, :, slot % 8], po.v[first + i])
        b0, _ = orc.branch_range[p]
        for idx in range(po.n_prefix, len(po.kind)):
            b, t = b0 + po.branch[idx], po.step_of[idx]
            assert np.abs(kt[b, :, t, :] - po.k[idx]).max() < 1e-5
            assert np.array_equal(vt[b, :, t, :], po.v[idx])


@pytest.mark.parametrize("kernel_mode,fused", [(0, False), (0, True), (1, False)])
def test_bf16_kv_pools_hold_the_rounded_rotated_keys(kernel_mode, fused):
    """The bf16 pools themselves (not only the attention outputs computed from them): prefix and
    tail keys must be the bf16 rounding of the oracle's fp32-rotated keys - the same value, held
    in IEEE half format, which represents every bf16 value of the normal half range exactly -
    except where the kernels' fused multiply-add lands on the other side of a rounding tie: such
    elements may differ by one bf16 ulp and must be rare -, values must be the input values in
    the same format, through the 8-key interleave of the prefix pool.  Covers the 128-channel fill kernel and
    the fused append of the streaming kernel (mode 0), the two-call append kernel, and the
    element-wise fill kernel (mode 1)."""
    from paper_2604_26209_amd import binding as B
    _say(f"bf16 pool contents mode {kernel_mode} fused {fused}")
    wl = W.random_workload(52, dtype="bf16", hq=8, hkv=2, d=128, base=500000.0, t=10, p=3,
                           j_range=(1, 3), n_range=(1, 9), l_range=(1, 150), h_range=(0, 70))
    hip = H.run_hip(wl, poison_pools="zero", kernel_mode=kernel_mode, fused=fused)
    orc, res = H.run_oracle(wl, hip["inputs"])  # bf16 key cache
    bits = lambda x: x.view(torch.int16).cpu().numpy().view(np.uint16)
    kp, vp, kt, vt = [bits(x) for x in hip["pools"]]
    lay = hip["layout"]
    c = lay.counts()
    NP, T, Hkv, D = int(c[B.HPD_C_N_PREFIX_SLOTS]), wl.max_new, wl.n_kv_heads, wl.head_dim
    kp = kp.reshape(Hkv, NP, D)
    vp = vp.reshape(Hkv, NP // 8, D, 8)
    kt = kt.reshape(wl.n_branches, Hkv, T, D)
    vt = vt.reshape(wl.n_branches, Hkv, T, D)
    as_bits = lambda a: (np.ascontiguousarray(a, dtype=np.float32).view(np.uint32) >> 16).astype(np.uint16)
    seg_off = B.hpd_layout_query(lay, B.HPD_Q_SEG_OFF)
    n_keys = n_off = 0

    def check_k(got_half, want_f32):
        # a key element is the bf16-rounded rotated key in IEEE half format: exact where the
        # value is a normal half (|k| >= 2^-14), within 2^-24 below that
        nonlocal n_keys, n_off
        want_f32 = np.ascontiguousarray(want_f32, dtype=np.float32)
        assert not np.any(want_f32.view(np.uint32) & 0xFFFF)
        got_f32 = np.ascontiguousarray(got_half).view(np.float16).astype(np.float32)
        normal = np.abs(want_f32) >= 2.0 ** -13
        assert not np.any(got_f32[normal].view(np.uint32) & 0xFFFF), "a stored key is not a bf16 value"
        diff = np.abs(as_bits(got_f32[normal]).astype(np.int32) - as_bits(want_f32[normal]).astype(np.int32))
        if diff.size:
            assert diff.max() <= 1, "a stored key is more than one bf16 ulp from the rounded oracle key"
        small = ~normal
        assert np.all(np.abs(got_f32[small] - want_f32[small]) <= 2.0 ** -24 + np.abs(want_f32[small]) * 2.0 ** -7)
        n_keys += diff.size
        n_off += int((diff != 0).sum())

    def check_v(got_half, want_f32):
        # a value element is the caller's bf16 value in half format: the same value wherever it
        # is a normal half, within 2^-24 below
        want_f32 = np.ascontiguousarray(want_f32, dtype=np.float32)
        got_f32 = np.ascontiguousarray(got_half).view(np.float16).astype(np.float32)
        normal = np.abs(want_f32) >= 2.0 ** -13
        assert np.array_equal(got_f32[normal], want_f32[normal])
        assert np.all(np.abs(got_f32[~normal] - want_f32[~normal]) <= 2.0 ** -24)

    for p, po in orc.prompts.items():
        segs = [(p, 0, po.h)]
        run = po.h
        for j, d in enumerate(range(wl.doc_ptr[p], wl.doc_ptr[p + 1])):
            segs.append((wl.n_prompts + d, run, po.doc_lens[j]))
            run += po.doc_lens[j]
        for sid, first, n in segs:
            for i in range(n):
                slot = seg_off[sid] + i
                check_k(kp[:, slot, :], po.k[first + i])
                check_v(vp[:, slot // 8, :, slot % 8], po.v[first + i])
            # the V padding behind the segment is zero (masked keys must contribute 0 * V = 0)
            for slot in range(seg_off[sid] + n, -(-(seg_off[sid] + n) // 32) * 32):
                assert not vp[:, slot // 8, :, slot % 8].any()
        b0, _ = orc.branch_range[p]
        for idx in range(po.n_prefix, len(po.kind)):
            b, t = b0 + po.branch[idx], po.step_of[idx]
            check_k(kt[b, :, t, :], po.k[idx])
            check_v(vt[b, :, t, :], po.v[idx])
    print(f"bf16 pools: {n_off} of {n_keys} stored key elements one ulp from the rounded oracle key "
          f"({n_off / n_keys:.2e})")
    assert n_off <= 2e-3 * n_keys


def test_error_paths_on_device_layout():
    from paper_2604_26209_amd import binding as B
    wl = W.config(1)
    lay = B.layout_from_workload(wl)
    with pytest.raises(B.HpdError):
        B.hpd_rope_positions(lay, wl.max_new, torch.zeros(4, dtype=torch.int32, device="cuda"))
    with pytest.raises(B.HpdError):
        B.hpd_rope_positions(lay, -1, torch.zeros(4, dtype=torch.int32, device="cuda"))
    with pytest.raises(B.HpdError):
        B.hpd_kv_append(lay, 0, None, None, None, None)
    with pytest.raises(B.HpdError):
        B.hpd_set_kernel_mode(lay, 2)  # fp32 / D=64 has no MFMA path
    x = torch.zeros(8, device="cuda")
    with pytest.raises(B.HpdError):
        B.hpd_prefill_attention(lay, None, x, x, x)
