"""GPU parity: the HIP library, called through its C ABI, against the CPU oracle
on the same seeded inputs, element by element.

Bars (from the benchmark contract): adversary masks and statuses bit-exact;
decoded sums within relative L2 1e-5 (repetition) / 1e-4 (cyclic) of the fp64
oracle on the SAME received messages; encoded messages within relative L2 1e-6
per node of the oracle's fp64 messages (the wire is fp32: one rounding is
6e-8); repetition copies bit-identical within a group."""
import os
import subprocess
import sys

import numpy as np
import pytest
import torch

from oracle import draco_oracle as o
from paper_1803_09877_amd import binding as B
from paper_1803_09877_amd import synth
from paper_1803_09877_amd.runner import Case

pytestmark = pytest.mark.gpu

TOL_MSG = 1e-6
TOL_SUM = {"rep": 1e-5, "cyc": 1e-4}


def rel_l2(a, b):
    a = np.asarray(a, dtype=np.float64)
    b = np.asarray(b, dtype=np.float64)
    nb = np.linalg.norm(b)
    return float(np.linalg.norm(a - b) / (nb if nb > 0 else 1.0))


def max_abs_err(a, b):
    """Largest element-wise deviation (a norm can hide a handful of wrong coordinates)."""
    return float(np.max(np.abs(np.asarray(a, dtype=np.float64) - np.asarray(b, dtype=np.float64)), initial=0.0))


def assert_message_close(zg, zo, ulps, what):
    """Every element of a message within `ulps` fp32 half-ulps of the row's largest entry:
    the encoders accumulate in fp64 (cyclic) or add r fp32 terms (repetition) and round once."""
    assert rel_l2(zg, zo) <= TOL_MSG, what
    bound = ulps * 2.0 ** -24 * float(np.max(np.abs(zo), initial=0.0))
    assert max_abs_err(zg, zo) <= bound, (what, max_abs_err(zg, zo), bound)


def assert_sum_close(ug, uo, tol, what):
    """Relative L2 and, element by element, within tol of the largest entry of the sum."""
    assert rel_l2(ug, uo) <= tol, (what, rel_l2(ug, uo))
    bound = tol * float(np.max(np.abs(uo), initial=0.0))
    assert max_abs_err(ug, uo) <= bound, (what, max_abs_err(ug, uo), bound)


WIDE = {"f32": (48, o.TAU_H_WIDE), "bf16": (33, o.TAU_H_BF16), "i8": (31.98, o.TAU_H_I8)}   # bits carried, threshold


def second_word_values(hi, lo, second):
    """fp64 values of a second-word slab (torch) next to its first words (numpy fp32): the stored
    number itself, or what an 8-bit code stands for at that first word."""
    if second == "i8":
        return o.residual_from_code8(hi, lo.cpu().numpy())
    return lo.double().cpu().numpy()


def wl(code, P, s, d, attacks=(), placement="any", sigma=1.0, seed=0):
    return synth.Workload(name=f"{code}_{P}_{s}_{d}", code=code, P=P, s=s, d=d, sigma=sigma,
                          attacks=tuple(attacks), placement=placement, seed=synth.SEED_BASE + 1000 + seed)


def oracle_encode(c: Case):
    G = c.G[:, :c.w.d].cpu().numpy()
    if c.w.code == "rep":
        return o.encode_repetition(G, c.w.s)
    return o.encode_cyclic(G, c.w.s)


def oracle_decode(c: Case, R_host):
    if c.w.code == "rep":
        return o.decode_repetition(R_host, c.w.s)
    return o.decode_cyclic(R_host, c.f.cpu().numpy(), c.w.s, c.w.d)


def run_and_check(w, extra_edit=None, expect_status=0, check_true_sum=None):
    print(f"case {w.name} P={w.P} s={w.s} d={w.d} attacks={w.attacks} seed={w.seed}", flush=True)
    c = Case(w)
    try:
        c.Z.fill_(float("nan"))                      # anything the encoder fails to write shows up
        c.encode()
        torch.cuda.synchronize()
        Zg = c.Z[:, :c.mlen].cpu().numpy()
        Zo = oracle_encode(c)
        assert Zg.shape == Zo.shape
        ulps = 2 * w.r if w.code == "rep" else 2
        for j in range(w.P):
            assert_message_close(Zg[j], Zo[j], ulps, f"message {j}")
        if c.ld_m > c.mlen:                           # padding untouched
            assert torch.isnan(c.Z[:, c.mlen:]).all()
        if w.code == "rep":
            r = w.r
            for j in range(w.P):
                assert np.array_equal(Zg[j].view(np.uint32), Zg[(j // r) * r].view(np.uint32))
        c.receive()
        if extra_edit is not None:
            extra_edit(c)
        R_host = c.R[:, :c.mlen].cpu().numpy()
        uo, mo, so = oracle_decode(c, R_host)
        # the cyclic decoder has two forms: phi and b on the device (default) and on the host
        for hostphi in ((False, True) if w.code == "cyc" else (False,)):
            c.u.fill_(float("nan"))
            mask, status = c.decode(hostphi=hostphi)
            torch.cuda.synchronize()
            assert status == so == expect_status, hostphi
            assert np.array_equal(mask, mo), hostphi
            if expect_status == 0:
                if extra_edit is None:
                    assert np.array_equal(mask, c.expected_mask())
                ug = c.u[:w.d].cpu().numpy()
                assert np.isfinite(ug).all()
                assert_sum_close(ug, uo, TOL_SUM[w.code], hostphi)
                if check_true_sum is not None:               # Definition 2, end to end, up to the fp32 wire
                    ref = c.G[:, :w.d].double().sum(0).cpu().numpy()
                    assert rel_l2(ug, ref) <= check_true_sum
            if c.u.numel() > w.d:
                assert torch.isnan(c.u[w.d:]).all()
        return c
    finally:
        c.close()


# ----------------------------------------------------------- repetition -----
def test_rep_config0_exact_recipe():
    run_and_check(synth.WORKLOADS[0], check_true_sum=1e-6)


@pytest.mark.parametrize("P,s,d,attacks,placement", [
    (3, 1, 1, ("noise",), "any"),
    (3, 1, 3, ("signflip",), "any"),
    (6, 1, 1023, ("constant",), "any"),
    (15, 1, 4097, ("noise",), "any"),
    (15, 2, 10_007, ("signflip", "noise"), "distinct_groups"),
    (15, 2, 10_007, ("signflip", "noise"), "any"),
    (45, 2, 70_001, ("signflip", "signflip"), "distinct_groups"),
    (6, 0, 5000, (), "any"),
    (21, 3, 3333, ("noise", "constant", "signflip"), "any"),
    (15, 7, 2050, ("noise",) * 7, "any"),
    (17, 8, 2051, ("noise",) * 8, "any"),             # r = 17: generic path
    (34, 8, 777, ("signflip", "noise", "constant"), "any"),
    (66, 1, 555, ("noise",), "any"),                   # more than 64 nodes: second mask word
    (255, 2, 300, ("noise", "signflip"), "distinct_groups"),
    (256, 0, 1030, (), "any"),                         # the largest P the library takes (r = 1: plain sum)
])
def test_rep_parity(P, s, d, attacks, placement):
    for seed in range(2):
        run_and_check(wl("rep", P, s, d, attacks, placement, seed=seed), check_true_sum=1e-6)


@pytest.mark.parametrize("kind", ["one_ulp", "nan", "neg_zero", "last_coord"])
def test_rep_bit_level_adversaries(kind):
    P, s, d = 15, 2, 5003

    def edit(c):
        j = 7
        if kind == "one_ulp":
            x = c.R[j, 1234:1235].view(torch.int32)
            x += 1
        elif kind == "nan":
            c.R[j, 77] = float("nan")
        elif kind == "neg_zero":
            c.R[:, 500] = 0.0
            c.R[j, 500] = -0.0
        elif kind == "last_coord":
            c.R[j, d - 1] += 1.0
    c = run_and_check(wl("rep", P, s, d), extra_edit=edit)


def test_rep_more_than_s_liars_is_reported():
    def edit(c):
        for j in (0, 2, 4):
            c.R[j, :c.mlen] = float(j + 1)
    run_and_check(wl("rep", 10, 2, 999), extra_edit=edit, expect_status=B.NO_MAJORITY)


@pytest.mark.parametrize("code,d", [("rep", 3001), ("cyc", 3001), ("cyc", 300_001)])
def test_a_failed_decode_leaves_no_state_behind(code, d):
    """A decode that reports too many adversaries, then a good one on the same plan: the
    second is as if the first had never run (flag words, scratch and, on the longer rows, which are
    not split over the nodes, speculation state)."""
    P, s = (10, 2) if code == "rep" else (9, 2)
    w = wl(code, P, s, d, ("signflip",))
    c = Case(w)
    try:
        c.encode()
        c.receive()
        good = c.R.clone()
        for j in (0, 2, 4) if code == "rep" else (0, 3, 6):
            c.R[j, :c.mlen] = float(j + 1) if code == "rep" else torch.randn(c.mlen, device=c.device) * 100
        mask, status = c.decode()
        assert status == (B.NO_MAJORITY if code == "rep" else B.LOCATE_FAILED)
        c.R.copy_(good)
        uo, mo, so = oracle_decode(c, good[:, :c.mlen].cpu().numpy())
        for _ in range(2):
            c.u.fill_(float("nan"))
            mask, status = c.decode()
            torch.cuda.synchronize()
            assert status == B.OK == so and np.array_equal(mask, mo) and np.array_equal(mask, c.expected_mask())
            assert rel_l2(c.u[:d].cpu().numpy(), uo) <= TOL_SUM[code]
    finally:
        c.close()


def test_rep_async_form_and_determinism():
    w = wl("rep", 45, 2, 123_457, ("signflip", "signflip"), "distinct_groups")
    c = Case(w)
    try:
        c.encode()
        c.receive()
        mask_dev = torch.zeros(4, dtype=torch.int64, device=c.device)
        status_dev = torch.full((1,), -7, dtype=torch.int32, device=c.device)
        outs = []
        for _ in range(2):
            c.u.zero_()
            c.plan.decode_repetition_async(c.R, c.u, mask_dev, status_dev)
            torch.cuda.synchronize()
            outs.append((c.u.clone(), mask_dev.clone(), int(status_dev.item())))
        assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][1], outs[1][1])
        assert outs[0][2] == 0
        m, st = c.decode()
        words = B.bool_to_mask(m, w.P)
        assert int(mask_dev[0].item()) == int(words[0].astype(np.int64))
        assert np.array_equal(m, c.expected_mask())
    finally:
        c.close()


# --------------------------------------------------------------- cyclic -----
@pytest.mark.parametrize("P,s,d,attacks,placement,sigma,e2e", [
    (4, 1, 2, ("signflip",), "any", 1.0, 1e-5),
    (4, 1, 1, ("offset",), "any", 1.0, 1e-5),
    (5, 2, 1001, ("noise", "offset"), "any", 1.0, 1e-5),           # P = 2s+1: every node holds everything
    (6, 0, 4099, (), "any", 1.0, 1e-5),
    (15, 2, 40_000, ("offset", "offset"), "any", 1.0, 1e-5),
    (15, 2, 40_003, ("offset", "signflip"), "adjacent_pair", 1.0, 1e-5),
    (15, 2, 40_002, ("noise",), "any", 1.0, 1e-5),
    (15, 2, 8191, (), "any", 1.0, 1e-5),
    (45, 3, 70_001, ("noise", "signflip", "noise"), "adjacent_pair", 1e-2, 2e-3),
    (45, 3, 70_002, ("signflip",), "any", 1e-2, 2e-3),
    (45, 1, 9_999, ("noise",), "any", 1e-2, 1e-4),
    (15, 7, 6_001, ("noise", "signflip", "offset", "constant", "noise", "signflip", "offset"), "any", 1.0, 1e-5),
    (20, 8, 3_001, ("noise", "signflip", "offset"), "any", 1.0, 1e-4),   # r = 17
    (23, 9, 2_051, ("noise", "signflip"), "any", 1.0, 1e-4),             # r = 19
    (24, 10, 1_031, ("noise",) * 10, "any", 1.0, 1e-4),                  # r = 21: widest register window
    (30, 11, 1_030, ("signflip", "noise"), "any", 1.0, 1e-3),            # r = 23: the LDS-ring encoder
    (40, 16, 515, ("noise",) * 5, "any", 1.0, None),                     # r = 33: largest s of the device locator
    (70, 2, 2_001, ("noise", "signflip"), "any", 1.0, None),       # second mask word
    (256, 1, 301, ("noise",), "any", 1.0, 1e-3),                   # the largest P the library takes
    (128, 2, 999, ("signflip", "noise"), "any", 1.0, None),        # wide dynamic range of W
    (200, 3, 500, ("noise", "noise"), "any", 1.0, None),           # the fp32 wire drowns the sum here; parity still holds
    # the constant adversary (Sec. 4, "Adversarial Attack Models") on wide windows and many nodes
    (45, 5, 30_000, ("constant",) * 5, "any", 1e-2, None),
    (45, 5, 30_001, ("constant", "signflip", "constant", "noise", "constant"), "any", 1e-2, None),
    (50, 7, 8_001, ("constant",) * 7, "any", 1.0, None),
    (50, 7, 8_000, ("constant", "constant", "noise"), "adjacent_pair", 1e-2, None),
    (63, 7, 5_003, ("constant",) * 7, "any", 1e-2, None),
    (40, 4, 12_001, ("constant",) * 4, "any", 1.0, None),
    (60, 6, 6_001, ("constant", "offset", "constant", "constant"), "any", 1e-2, None),
])
def test_cyc_parity(P, s, d, attacks, placement, sigma, e2e):
    for seed in range(2):
        run_and_check(wl("cyc", P, s, d, attacks, placement, sigma, seed=seed), check_true_sum=e2e)


def test_cyc_more_than_s_adversaries_is_reported():
    def edit(c):
        g = torch.Generator(device=c.device)
        g.manual_seed(5)
        for j in (0, 3, 6):
            c.R[j, :c.mlen] = torch.randn(c.mlen, generator=g, device=c.device) * 100
    run_and_check(wl("cyc", 9, 2, 4001), extra_edit=edit, expect_status=B.LOCATE_FAILED)


@pytest.mark.parametrize("bad", ["inf", "nan", "two_nodes", "with_other_liar"])
def test_cyc_nonfinite_messages_are_flagged_and_survived(bad):
    """A node that sends NaN or Inf is flagged outright and the sum is still recovered
    (it is one of the at most s adversaries); more broken nodes than s is reported."""
    def edit(c):
        if bad == "inf":
            c.R[2, 10] = float("inf")
        elif bad == "nan":
            c.R[7, c.mlen - 1] = float("nan")
        elif bad == "two_nodes":
            c.R[2, 10] = float("inf")
            c.R[3, 11] = float("nan")
        else:
            c.R[2, 10] = float("nan")
            c.R[5, :c.mlen] *= -100.0
    c = run_and_check(wl("cyc", 9, 2, 4001), extra_edit=edit, check_true_sum=1e-5)


@pytest.mark.parametrize("wire", ["one", "i8", "bf16", "f32"])
@pytest.mark.parametrize("P,s,d", [(15, 2, 8_001), (45, 3, 20_000)])
def test_cyc_enormous_lies_are_located(P, s, d, wire):
    """Definition 2 bounds nothing an adversary sends: first words scaled by 1e2 .. 1e30 (the edge
    of fp32), alone or with an ordinary lie at another node hiding behind them, on every wire.
    Mask, status and sum as the oracle's on the same received words; both decoder forms."""
    w = wl("cyc", P, s, d, (), "any", 1e-2)
    c = Case(w, wide=False if wire == "one" else wire)
    tau = o.TAU_H if wire == "one" else WIDE[wire][1]
    try:
        c.encode()
        torch.cuda.synchronize()
        ref = c.G[:, :d].double().sum(0).cpu().numpy()
        g = torch.Generator(device=c.device)
        g.manual_seed(5)
        for it, mag in enumerate((1e2, 1e6, 1e9, 1e12, 1e20, 1e30)):
            c.receive()
            big, small = (3 + it) % P, (4 + 5 * it) % P
            scale = float(c.Z[:, :c.mlen].abs().max())
            if it % 2 == 0:
                c.R[big, :c.mlen] = torch.randn(c.mlen, generator=g, device=c.device) * min(mag * scale, 1e37)
            else:
                c.R[big, :c.mlen] *= -mag
            liars = {big}
            if s >= 2 and small != big:
                c.R[small, :c.mlen] += 10.0 * scale * torch.randn(c.mlen, generator=g, device=c.device)
                liars.add(small)
            Rhi = c.R[:, :c.mlen].cpu().numpy()
            Rw = Rhi.astype(np.float64) + (second_word_values(Rhi, c.Rlo[:, :c.mlen], wire) if wire != "one" else 0.0)
            uo, mo, so = o.decode_cyclic(Rw, c.f.cpu().numpy(), s, d, tau_h=tau)
            assert so == o.OK and set(np.flatnonzero(mo)) == liars, (mag, np.flatnonzero(mo), liars)
            for hostphi in ((False, True) if wire == "one" else (False,)):
                c.u.fill_(float("nan"))
                mask, status = c.decode(hostphi=hostphi)
                torch.cuda.synchronize()
                assert status == B.OK and np.array_equal(mask, mo), (mag, hostphi, status, np.flatnonzero(mask))
                ug = c.u[:d].cpu().numpy()
                assert_sum_close(ug, uo, 1e-4 if wire == "one" else 1e-6, (mag, hostphi))
                assert rel_l2(ug, ref) <= (2e-3 if wire == "one" and P >= 32 else 1e-4)
    finally:
        c.close()


def test_cyc_more_enormous_lies_than_s_is_reported():
    def edit(c):
        for j in (1, 4, 6):
            c.R[j, :c.mlen] *= 1e28
    run_and_check(wl("cyc", 9, 2, 4001), extra_edit=edit, expect_status=B.LOCATE_FAILED)


def test_cyc_more_broken_messages_than_s_is_reported():
    def edit(c):
        for j in (1, 4, 6):
            c.R[j, 3 + j] = float("nan")
    run_and_check(wl("cyc", 9, 2, 4001), extra_edit=edit, expect_status=B.LOCATE_FAILED)


@pytest.mark.parametrize("P,s,d", [(45, 3, 2_001), (100, 2, 515), (256, 16, 301)])
def test_cyc_every_message_broken_is_reported_not_overrun(P, s, d):
    """A diverged step: all P messages hold NaN (far more broken nodes than the locator's
    work arrays of 2*16 entries).  Both decoder forms report LOCATE_FAILED with every node
    flagged, as the oracle does."""
    def edit(c):
        c.R[:, 1] = float("nan")
    run_and_check(wl("cyc", P, s, d), extra_edit=edit, expect_status=B.LOCATE_FAILED)


def test_cyc_async_form_needs_no_host_value():
    w = wl("cyc", 45, 3, 90_001, ("noise", "signflip", "noise"), "adjacent_pair", sigma=1e-2)
    c = Case(w)
    try:
        c.encode()
        c.receive()
        mask_dev = torch.zeros(4, dtype=torch.int64, device=c.device)
        status_dev = torch.full((1,), -7, dtype=torch.int32, device=c.device)
        c.u.zero_()
        c.plan.decode_cyclic_async(c.R, c.f, c.u, mask_dev, status_dev)
        torch.cuda.synchronize()
        u_async = c.u.clone()
        m, st = c.decode()
        assert st == 0 == int(status_dev.item())
        assert int(mask_dev[0].item()) == int(B.bool_to_mask(m, w.P)[0].astype(np.int64))
        assert np.array_equal(m, c.expected_mask())
        assert torch.equal(u_async, c.u)
        mh, sth = c.decode(hostphi=True)
        assert sth == 0 and np.array_equal(mh, m)
        assert rel_l2(c.u[:w.d].cpu().numpy(), u_async[:w.d].cpu().numpy()) <= 1e-6
    finally:
        c.close()


def test_cyc_speculative_single_pass_decode():
    """A plan speculates when its previous decode was clean.  Sequence on one plan: clean,
    clean, two liars, two liars, clean, clean -- every result against the oracle, the clean
    speculated ones bit-identical to the two-pass result, and the second pass then costs
    next to nothing."""
    w = wl("cyc", 45, 3, 2_000_001, (), "any", 1e-2)
    c = Case(w)
    ref = Case(w)
    ref.plan.set_speculation(False)
    try:
        c.encode()
        f = c.f.cpu().numpy()
        c.plan.set_timing(16)
        liars = [(10, "signflip"), (11, "noise")]
        for step, adv in enumerate([[], [], liars, liars, [], []]):
            c.R = c.Z.clone()
            synth.apply_attacks(c.R, c.mlen, adv, w.seed + step)
            ref.R = c.R
            c.u.fill_(float("nan"))
            mask, status = c.decode()
            ref.u.fill_(float("nan"))
            mask_ref, status_ref = ref.decode()
            torch.cuda.synchronize()
            proj_ms, _ = c.plan.kernel_time(B.KIND_PROJECT)
            reco_ms, _ = c.plan.kernel_time(B.KIND_RECOMBINE)
            uo, mo, so = o.decode_cyclic(c.R[:, :c.mlen].cpu().numpy(), f, w.s, w.d)
            assert status == status_ref == so == 0
            assert np.array_equal(mask, mo) and np.array_equal(mask_ref, mo)
            assert sorted(np.flatnonzero(mask)) == sorted(j for j, _ in adv)
            assert rel_l2(c.u[:w.d].cpu().numpy(), uo) <= 1e-4
            assert torch.equal(c.u[:w.d], ref.u[:w.d]), step       # same bits with and without speculation
            assert torch.isnan(c.u[w.d:]).all()
            speculated_and_clean = not adv and (step == 0 or step == 1 or step == 5)
            print(f"   step {step}: liars {len(adv)}  project {proj_ms:.3f} ms  recombine {reco_ms:.3f} ms", flush=True)
            if speculated_and_clean:
                assert reco_ms < 0.25 * proj_ms
            else:
                assert reco_ms > 0.5 * proj_ms
    finally:
        c.close()
        ref.close()


@pytest.mark.parametrize("d", [150_001, 400_001, 600_001, 1_100_001])
@pytest.mark.parametrize("second", [False, "i8", "bf16", "f32"])
def test_cyc_speculation_over_a_random_run_of_steps(second, d):
    """Twenty steps on one plan with the adversaries changing at random (none, some, enormous
    ones that cost the locator extra passes, a broken message): the speculating plan and one
    that never speculates write the same bits, masks and statuses at every step, on every wire: on rows
    split over the nodes (no speculation), and with one and two float4 per lane, where a clean
    step after a clean one leaves the second pass out."""
    P, s = 33, 3
    w = wl("cyc", P, s, d, (), "any", 1e-2)
    c = Case(w, wide=second)
    ref = Case(w, wide=second)
    ref.plan.set_speculation(False)
    rng = np.random.default_rng(77)
    c.plan.set_timing(32)
    ref.plan.set_timing(32)
    before, skipped = True, 0
    try:
        c.encode()
        ref.Z, ref.Zlo = c.Z, c.Zlo
        for step in range(20):
            c.receive()
            k = int(rng.choice([0, 0, 0, 1, 2, 3]))
            liars = sorted(rng.choice(P, size=k, replace=False).tolist())
            for j in liars:
                kind = int(rng.integers(0, 4))
                if kind == 0:
                    c.R[j, :c.mlen] *= -100.0
                elif kind == 1:
                    c.R[j, :c.mlen] *= float(10.0 ** rng.integers(3, 30))
                elif kind == 2:
                    c.R[j, :c.mlen] += 1e3
                else:
                    c.R[j, int(rng.integers(0, c.mlen))] = float("nan")
            ref.R, ref.Rlo = c.R, c.Rlo
            c.u.fill_(float("nan"))
            ref.u.fill_(float("nan"))
            mask, status = c.decode()
            mask_ref, status_ref = ref.decode()
            torch.cuda.synchronize()
            assert status == status_ref == 0, (step, liars)
            assert np.array_equal(mask, mask_ref) and sorted(np.flatnonzero(mask)) == liars, (step, liars)
            assert torch.equal(c.u[:d].view(torch.int32), ref.u[:d].view(torch.int32)), (step, liars)
            assert torch.isfinite(c.u[:d]).all() and torch.isnan(c.u[d:]).all()
            one_pass = c.plan.kernel_times(B.KIND_RECOMBINE)[-1] < 0.7 * ref.plan.kernel_times(B.KIND_RECOMBINE)[-1]
            if d > 150_001:
                assert one_pass == (before and not liars), (step, liars)
            before = not liars
            skipped += one_pass
        assert skipped > 0 or d == 150_001
    finally:
        c.close()
        ref.close()


@pytest.mark.parametrize("P,s,d,attacks,sigma,seed", [
    (15, 2, 10_007, ("offset", "noise"), 1.0, 0),
    (45, 3, 70_002, ("signflip", "noise", "noise"), 1e-2, 0x9E3779B97F4A7C15),
    (9, 4, 515, ("noise",) * 4, 1.0, 2**64 - 1),
    (45, 3, 40_000, (), 1e-2, 12345),
])
def test_cyc_generated_projection_vector(P, s, d, attacks, sigma, seed):
    """f_dev = NULL: the projection kernel draws f itself from (seed, index).  The oracle
    draws the same vector with its own implementation of the generator and decodes with it."""
    w = wl("cyc", P, s, d, attacks, "any", sigma)
    print(f"case {w.name} generated f, seed={seed}", flush=True)
    c = Case(w)
    try:
        c.encode()
        c.receive()
        torch.cuda.synchronize()
        R_host = c.R[:, :c.mlen].cpu().numpy()
        fo = o.projection_vector((d + 1) // 2, seed)
        uo, mo, so = o.decode_cyclic(R_host, fo, s, d)
        assert so == o.OK and np.array_equal(mo, c.expected_mask())
        for form in ("device", "host"):
            c.plan.set_projection_seed(seed)           # the first decode after this call uses exactly `seed`
            c.u.fill_(float("nan"))
            fn = c.plan.decode_cyclic if form == "device" else c.plan.decode_cyclic_hostphi
            mask, status = fn(c.R, None, c.u)
            torch.cuda.synchronize()
            assert status == B.OK and np.array_equal(mask, mo), form
            assert rel_l2(c.u[:d].cpu().numpy(), uo) <= TOL_SUM["cyc"], form
        # the generated vector is the one the host routine reports: feeding that one in by
        # pointer gives the same projections, hence bit-identical output
        u_gen = c.u.clone()
        f_dev = torch.from_numpy(c.plan.projection_vector(seed)).to(c.device)
        mask2, _ = c.plan.decode_cyclic_hostphi(c.R, f_dev, c.u)
        torch.cuda.synchronize()
        assert np.array_equal(mask2, mo)
        assert rel_l2(c.u[:d].cpu().numpy(), u_gen[:d].cpu().numpy()) <= 1e-6
        # another seed: another f, same answer
        c.plan.set_projection_seed(seed ^ 0x5555)
        mask3, status3 = c.plan.decode_cyclic(c.R, None, c.u)
        torch.cuda.synchronize()
        assert status3 == B.OK and np.array_equal(mask3, mo)
        assert rel_l2(c.u[:d].cpu().numpy(), uo) <= TOL_SUM["cyc"]
    finally:
        c.close()


@pytest.mark.parametrize("P,s,d,attacks,sigma", [
    (5, 1, 1, ("noise",), 1.0),
    (5, 2, 7, ("signflip", "noise"), 1.0),
    (15, 2, 10_007, ("offset", "offset"), 1.0),
    (15, 2, 4096, (), 1.0),
    (45, 3, 30_001, ("noise", "signflip", "noise"), 1e-2),
    (9, 4, 2050, ("noise",) * 4, 1.0),
    (15, 7, 1030, ("signflip",) * 7, 1.0),
    (17, 8, 515, ("noise",) * 8, 1.0),
    (21, 10, 2_050, ("noise", "signflip"), 1.0),       # widest register window
    (25, 11, 515, ("noise",) * 3, 1.0),                # window wider than the register kernels: per-node path
    (66, 1, 777, ("noise",), 1.0),
])
def test_cyc_unpacked_wire(P, s, d, attacks, sigma):
    """Sec. 3's cyclic code on the real gradients (messages of d complex entries): encoder
    against the oracle's Z = G W, decoder (device and host locator) against the oracle on
    the same received messages, and Definition 2 end to end."""
    run_unpacked(wl("cyc", P, s, d, attacks, "any", sigma))


def run_unpacked(w, e2e=None):
    P, s, d, attacks = w.P, w.s, w.d, w.attacks
    print(f"case {w.name} unpacked attacks={attacks} seed={w.seed}", flush=True)
    c = Case(w, unpacked=True)
    try:
        assert c.mlen == 2 * d and c.f.numel() == d
        c.Z.fill_(float("nan"))
        c.encode()
        torch.cuda.synchronize()
        Zg = c.Z[:, :c.mlen].cpu().numpy()
        Zo = o.encode_cyclic_unpacked(c.G[:, :d].cpu().numpy(), s)
        for j in range(P):
            assert rel_l2(Zg[j], Zo[j]) <= TOL_MSG, f"message {j}"
        if c.ld_m > c.mlen:
            assert torch.isnan(c.Z[:, c.mlen:]).all()
        c.receive()
        R_host = c.R[:, :c.mlen].cpu().numpy()
        uo, mo, so, resid = o.decode_cyclic_unpacked(R_host, c.f.cpu().numpy(), s)
        assert so == o.OK and np.array_equal(mo, c.expected_mask())
        forms = ((False, True) if s <= 16 else (True,))
        for hostphi in forms:
            c.u.fill_(float("nan"))
            mask, status = c.decode(hostphi=hostphi)
            torch.cuda.synchronize()
            assert status == B.OK and np.array_equal(mask, mo), hostphi
            ug = c.u[:d].cpu().numpy()
            assert np.isfinite(ug).all()
            assert rel_l2(ug, uo) <= TOL_SUM["cyc"], hostphi
            if c.u.numel() > d:
                assert torch.isnan(c.u[d:]).all()
        if s <= 16:   # stream-ordered form and the generated f
            mask_dev = torch.zeros(4, dtype=torch.int64, device=c.device)
            status_dev = torch.full((1,), -7, dtype=torch.int32, device=c.device)
            c.plan.set_projection_seed(99)
            c.u.fill_(float("nan"))
            c.plan.decode_cyclic_async(c.R, None, c.u, mask_dev, status_dev)
            torch.cuda.synchronize()
            assert int(status_dev.item()) == 0
            words = mask_dev.cpu().numpy().view(np.uint64)
            assert np.array_equal(B.mask_to_bool(words, P), mo)
            u2, m2, s2, _ = o.decode_cyclic_unpacked(R_host, o.projection_vector(d, 99), s)
            assert rel_l2(c.u[:d].cpu().numpy(), u2) <= TOL_SUM["cyc"]
        ref = c.G[:, :d].double().sum(0).cpu().numpy()     # Definition 2 up to the fp32 wire
        assert rel_l2(c.u[:d].cpu().numpy(), ref) <= (e2e if e2e is not None else (2e-3 if P >= 45 else 1e-4))
    finally:
        c.close()


@pytest.mark.parametrize("P,s,d", [(15, 2, 3001), (45, 3, 2048), (21, 10, 1030), (25, 11, 515)])
def test_cyc_unpacked_encode_node_is_bit_identical_to_the_all_node_form(P, s, d):
    w = wl("cyc", P, s, d)
    c = Case(w, unpacked=True)
    try:
        c.encode()
        r = w.r
        for node in range(P):
            Gn = c.G[[(node + t) % P for t in range(r)]].contiguous()
            z = torch.full((c.ld_m,), float("nan"), dtype=torch.float32, device=c.device)
            c.plan.encode_node(node, Gn, z)
            torch.cuda.synchronize()
            assert torch.equal(z[:c.mlen].view(torch.int32), c.Z[node, :c.mlen].view(torch.int32)), node
            assert torch.isnan(z[c.mlen:]).all()
    finally:
        c.close()


def test_cyc_unpacked_wire_rejects_what_it_does_not_support():
    w = wl("cyc", 9, 2, 100)
    c = Case(w, unpacked=True)
    try:
        lo = torch.zeros_like(c.Z)
        with pytest.raises(B.DracoError) as e:
            c.plan.encode_wide(c.G, c.Z, lo)
        assert e.value.status == B.EINVAL
        with pytest.raises(B.DracoError) as e:
            c.plan.decode_cyclic_wide(c.Z, lo, c.f, c.u)
        assert e.value.status == B.EINVAL
        with pytest.raises(B.DracoError) as e:                  # the wire is fixed once the plan is prepared
            c.plan.set_wire(B.WIRE_PACKED)
        assert e.value.status == B.EINVAL
        narrow = torch.zeros((9, 104), dtype=torch.float32, device=c.device)   # a packed-size slab is too short
        with pytest.raises(B.DracoError) as e:
            c.plan.encode(c.G, narrow)
        assert e.value.status == B.EALIGN
    finally:
        c.close()


def test_cyc_large_s_takes_the_host_form():
    # s = 17 > 16: the default entry point falls back to host phi; the async form refuses
    w = wl("cyc", 40, 17, 1_001, ("noise", "signflip", "offset"), "any")
    c = run_and_check(w)
    c2 = Case(w)
    try:
        mask_dev = torch.zeros(4, dtype=torch.int64, device=c2.device)
        status_dev = torch.zeros(1, dtype=torch.int32, device=c2.device)
        c2.encode()
        c2.receive()
        with pytest.raises(B.DracoError) as e:
            c2.plan.decode_cyclic_async(c2.R, c2.f, c2.u, mask_dev, status_dev)
        assert e.value.status == B.EINVAL
    finally:
        c2.close()


@pytest.mark.parametrize("P,s,d,attacks,placement,sigma", [
    (15, 2, 40_003, ("offset", "signflip"), "adjacent_pair", 1.0),
    (45, 3, 70_001, ("noise", "signflip", "noise"), "adjacent_pair", 1e-2),
    (45, 3, 70_002, (), "any", 1e-2),
    (45, 5, 30_000, ("noise", "signflip", "offset", "constant", "noise"), "any", 1e-2),
    (20, 8, 3_001, ("noise", "signflip", "offset"), "any", 1.0),
    (30, 9, 2_051, ("noise", "signflip"), "any", 1.0),
    (24, 10, 1_031, ("noise", "offset"), "any", 1.0),
    (30, 12, 1_030, ("noise",), "any", 1.0),                              # LDS-ring encoder
    (40, 17, 1_001, ("noise", "signflip"), "any", 1.0),                  # host phi fallback
])
@pytest.mark.parametrize("second", ["f32", "bf16", "i8"])
def test_cyc_wide_wire(P, s, d, attacks, placement, sigma, second):
    """Two-word wire: hi + lo carries the fp64 message to 48 bits (32 with a bfloat16 or an
    8-bit second word), so the decoded sum meets Definition 2 END TO END (against the true gradient sum)
    far inside the 1e-4 bar also at P = 45, where the one-word wire cannot."""
    run_wide(wl("cyc", P, s, d, attacks, placement, sigma), second)


def run_wide(w, second="f32", e2e=None):
    P = w.P
    print(f"wide case {w.name} second word {second} attacks={w.attacks} seed={w.seed}", flush=True)
    c = Case(w, wide=second)
    bits, tau = WIDE[second]
    try:
        c.Z.fill_(float("nan"))
        c.Zlo.fill_(77 if second == "i8" else float("nan"))
        c.encode()
        torch.cuda.synchronize()
        assert c.Zlo.dtype == {"f32": torch.float32, "bf16": torch.bfloat16, "i8": torch.int8}[second]
        Zhi = c.Z[:, :c.mlen].cpu().numpy()
        Zlo = second_word_values(Zhi, c.Zlo[:, :c.mlen], second)
        Zw = Zhi.astype(np.float64) + Zlo
        Zo = o.encode_cyclic(c.G[:, :w.d].cpu().numpy(), w.s)
        # hi + lo against the fp64 message: what the wire's bits allow, element by element, plus the
        # two sides' fp64 summation orders (W itself agrees to 1e-14)
        for j in range(P):
            slack = 2.0 ** -bits * np.abs(Zo[j]) + 2.0 ** -43 * np.abs(Zo[j]).max()
            assert (np.abs(Zw[j] - Zo[j]) <= slack).all(), j
        # the two words themselves against the oracle's wire: the same bits wherever the two fp64
        # messages round alike (they differ by 1e-16, so all but a handful of elements)
        hi_o, lo_o = o.two_word_wire(Zo, second)
        same_hi = Zhi.view(np.uint32) == hi_o.view(np.uint32)
        # (weights like 3 and -1.5 put many fp64 messages exactly on an fp32 tie, which the two
        # sides' 1e-15 then break differently: the first word is a correct rounding either way)
        assert (np.abs(Zhi.astype(np.float64) - Zo) <= 2.0 ** -24 * np.abs(Zo) * (1 + 2.0 ** -20) + 2.0 ** -43 * np.abs(Zo).max()).all()
        assert same_hi.mean() >= 0.8
        if second != "f32":     # (an fp32 residual resolves the 1e-16 itself: covered by the bound above)
            # (a message that IS an fp32 number leaves a residual of rounding noise, 1e-16 of either sign)
            same_lo = (Zlo == lo_o) | (np.abs(Zlo - lo_o) <= 2.0 ** -43 * np.abs(Zo).max())
            assert same_lo[same_hi].mean() >= 0.99
        if c.ld_m > c.mlen:
            assert torch.isnan(c.Z[:, c.mlen:]).all()
            pad = c.Zlo[:, c.mlen:]
            assert (pad == 77).all() if second == "i8" else torch.isnan(pad.float()).all()
        c.receive()
        c.u.fill_(float("nan"))
        mask, status = c.decode()
        torch.cuda.synchronize()
        Rhi = c.R[:, :c.mlen].cpu().numpy()
        Rw = Rhi.astype(np.float64) + second_word_values(Rhi, c.Rlo[:, :c.mlen], second)
        uo, mo, so = o.decode_cyclic(Rw, c.f.cpu().numpy(), w.s, w.d, tau_h=tau)
        assert status == so == 0
        assert np.array_equal(mask, mo) and np.array_equal(mask, c.expected_mask())
        ug = c.u[:w.d].cpu().numpy()
        assert_sum_close(ug, uo, 1e-6, second)
        ref = c.G[:, :w.d].double().sum(0).cpu().numpy()
        # fp32 output rounding is 6e-8; the 32-bit wire's own floor is W's growth times 2^-33
        assert rel_l2(ug, ref) <= (e2e if e2e is not None else {"f32": 1e-6, "bf16": 1e-5, "i8": 3e-5}[second])
        if c.u.numel() > w.d:
            assert torch.isnan(c.u[w.d:]).all()
    finally:
        c.close()


@pytest.mark.parametrize("P,s,d,size,second", [(15, 2, 20_001, 1e-9, "f32"), (45, 3, 30_000, 1e-8, "f32"),
                                                (9, 4, 4099, 1e-8, "f32"), (15, 2, 20_001, 5e-7, "bf16")])
def test_cyc_wide_wire_tells_tiny_lies_from_rounding(P, s, d, size, second):
    """On the two-word wire a lie of 1e-8 .. 1e-9 of the message size (far below an fp32
    ulp: the adversary edits the second word) is located, with the wide wire's threshold on
    both sides; the one-word threshold would wave it through.  With a bfloat16 second word the
    same at 5e-7, between that wire's threshold and the one-word one (at small P: the 2^9 between
    the two thresholds is less than the locator's own error growth at P = 45)."""
    w = wl("cyc", P, s, d, (), "any", 1.0)
    c = Case(w, wide=second)
    tau = o.TAU_H_WIDE if second == "f32" else o.TAU_H_BF16
    try:
        c.encode()
        c.receive()
        liars = [1, P - 1][:s]
        scale = float(c.Z[:, :c.mlen].abs().median())
        g = torch.Generator(device=c.device)
        g.manual_seed(9)
        for j in liars:
            lie = torch.randn(c.mlen, generator=g, device=c.device) * (size * scale)
            c.Rlo[j, :c.mlen] = (c.Rlo[j, :c.mlen].float() + lie).to(c.Rlo.dtype)
        Rw = c.R[:, :c.mlen].double().cpu().numpy() + c.Rlo[:, :c.mlen].double().cpu().numpy()
        f = c.f.cpu().numpy()
        uo, mo, so = o.decode_cyclic(Rw, f, s, d, tau_h=tau)
        assert so == o.OK and sorted(np.flatnonzero(mo)) == sorted(liars)
        _, m_loose, _ = o.decode_cyclic(Rw, f, s, d)                      # the one-word threshold sees nothing
        assert not m_loose.any()
        for fn in (c.plan.decode_cyclic_wide,):
            c.u.fill_(float("nan"))
            mask, status = fn(c.R, c.Rlo, c.f, c.u)
            torch.cuda.synchronize()
            assert status == B.OK and np.array_equal(mask, mo)
            assert rel_l2(c.u[:d].cpu().numpy(), uo) <= 1e-6
        ref = c.G[:, :d].double().sum(0).cpu().numpy()
        assert rel_l2(c.u[:d].cpu().numpy(), ref) <= (1e-6 if second == "f32" else 1e-5)
    finally:
        c.close()


@pytest.mark.parametrize("second", ["f32", "bf16", "i8"])
def test_cyc_wide_wire_survives_broken_and_hostile_words(second):
    """Two-word wire, s = 2: one node's FIRST word holds an Inf, another node's SECOND words are
    hostile -- NaN where the format has one, else the code 0x80 (which no encoder writes) under a
    sign-flipped first word.  Both are flagged, neither row reaches the sum; mask, status and sum
    as the oracle's on the same words."""
    w = wl("cyc", 9, 2, 4_001)
    c = Case(w, wide=second)
    try:
        c.encode()
        c.receive()
        c.R[2, 10] = float("inf")
        if second == "i8":
            c.Rlo[6, :c.mlen] = -128
            c.R[6, :c.mlen] *= -100.0
        else:
            c.Rlo[6, 5] = float("nan")
        Rhi = c.R[:, :c.mlen].cpu().numpy()
        Rw = Rhi.astype(np.float64) + second_word_values(Rhi, c.Rlo[:, :c.mlen], second)
        assert not np.isfinite(Rw[2]).all() and (second == "i8" or not np.isfinite(Rw[6]).all())
        with np.errstate(invalid="ignore"):
            uo, mo, so = o.decode_cyclic(Rw, c.f.cpu().numpy(), w.s, w.d, tau_h=WIDE[second][1])
        assert so == o.OK and sorted(np.flatnonzero(mo)) == [2, 6]
        for fn in (c.plan.decode_cyclic_wide,):
            c.u.fill_(float("nan"))
            mask, status = fn(c.R, c.Rlo, c.f, c.u)
            torch.cuda.synchronize()
            assert status == B.OK and np.array_equal(mask, mo)
            ug = c.u[:w.d].cpu().numpy()
            assert np.isfinite(ug).all()
            assert_sum_close(ug, uo, 1e-6, second)
        ref = c.G[:, :w.d].double().sum(0).cpu().numpy()
        assert rel_l2(ug, ref) <= 1e-5
    finally:
        c.close()


def test_cyc_determinism():
    w = wl("cyc", 15, 2, 100_003, ("offset", "offset"))
    c = Case(w)
    try:
        c.encode()
        z0 = c.Z.clone()
        c.encode()
        assert torch.equal(z0, c.Z)
        c.receive()
        outs = []
        for _ in range(2):
            c.u.zero_()
            m, st = c.decode()
            outs.append((c.u.clone(), m))
        assert torch.equal(outs[0][0], outs[1][0]) and np.array_equal(outs[0][1], outs[1][1])
    finally:
        c.close()


# ------------------------------------ the two sides end to end, nothing shared ----
@pytest.mark.parametrize("code,P,s,d,attacks,wire", [
    ("rep", 15, 2, 30_001, ("signflip", "offset"), "one"),
    ("cyc", 15, 2, 30_001, ("signflip", "offset"), "one"),
    ("cyc", 45, 3, 30_002, ("signflip", "constant", "offset"), "f32"),
    ("cyc", 45, 3, 30_002, ("signflip", "constant", "offset"), "bf16"),
    ("cyc", 45, 3, 30_002, ("signflip", "constant", "offset"), "i8"),
    ("cyc", 45, 5, 8_001, ("constant", "signflip", "constant", "signflip", "constant"), "i8"),
])
def test_both_sides_end_to_end_from_the_same_gradients(code, P, s, d, attacks, wire):
    """Nothing of the library's output enters the oracle here: from the SAME gradients the oracle
    encodes in fp64, puts its messages on its own model of the wire, applies the (deterministic)
    attacks and decodes; the library encodes, receives the same attacks and decodes.  Masks equal,
    sums within the code's tolerance of each other and of the true sum."""
    w = wl(code, P, s, d, attacks, "any", 1e-2 if code == "cyc" else 1.0)
    c = Case(w, wide=False if wire == "one" else wire)
    try:
        G = c.G[:, :d].cpu().numpy()
        f = c.f.cpu().numpy() if code == "cyc" else None
        # the oracle's side
        Zo = o.encode_repetition(G, s) if code == "rep" else o.encode_cyclic(G, s)
        if wire == "one":
            hi, lo, tau = Zo.astype(np.float32), 0.0, o.TAU_H
        else:
            hi, lo = o.two_word_wire(Zo, wire)
            tau = WIDE[wire][1]
        hi_t = torch.from_numpy(hi.copy())
        synth.apply_attacks(hi_t, hi.shape[1], c.adversaries, w.seed)          # edits the first word, as on the GPU
        Ro = hi_t.numpy().astype(np.float64) + lo if wire != "one" else hi_t.numpy()
        if code == "rep":
            uo, mo, so = o.decode_repetition(Ro, s)
        else:
            uo, mo, so = o.decode_cyclic(Ro, f, s, d, tau_h=tau)
        # the library's side
        c.encode()
        c.receive()
        c.u.fill_(float("nan"))
        mask, status = c.decode()
        torch.cuda.synchronize()
        assert status == so == 0
        assert np.array_equal(mask, mo) and np.array_equal(mask, c.expected_mask())
        ug = c.u[:d].cpu().numpy()
        tol = TOL_SUM[code]
        assert_sum_close(ug, uo, tol, wire)
        ref = G.astype(np.float64).sum(0)
        if not (code == "cyc" and wire == "one" and P >= 32):
            assert rel_l2(ug, ref) <= tol and rel_l2(uo, ref) <= tol
    finally:
        c.close()


# ------------------------------------------- workgroup footprint boundaries ----
@pytest.mark.parametrize("d", [255, 256, 257, 1023, 1025, 8191, 8192, 8193, 8449, 16385, 24577, 32767, 32768, 32769,
                               32768 + 8192 + 3, 65535, 65536, 65537, 3 * 32768 - 1, 3 * 32768 + 2049])
def test_lengths_around_the_footprint_windows(d):
    """A workgroup's wavefronts sit 32 KiB apart inside 128 KiB windows of a row (and a lane of the
    narrow-window cyclic encoder owns four pieces 8 KiB apart), so a row that ends near a piece, a
    wavefront stride or a window boundary leaves workgroups with some wavefronts inside the row and
    some outside: lengths one below, on and one above each boundary, for both codes, both packed
    cyclic encoders (rounds of rows; four pieces per lane) and all five wires."""
    run_and_check(wl("rep", 9, 1, d, ("noise",), "any"), check_true_sum=1e-6)
    run_and_check(wl("rep", 25, 2, d, ("signflip",), "any"), check_true_sum=1e-6)
    run_and_check(wl("cyc", 9, 1, d, ("noise",), "any"), check_true_sum=1e-5)
    run_and_check(wl("cyc", 33, 2, d, ("noise", "signflip"), "any", 1e-2))      # four pieces per lane
    run_wide(wl("cyc", 33, 3, d, ("noise", "offset", "signflip"), "any", 1e-2))
    run_wide(wl("cyc", 33, 3, d, ("noise", "offset", "signflip"), "any", 1e-2), "bf16")
    run_wide(wl("cyc", 33, 3, d, ("noise", "offset", "signflip"), "any", 1e-2), "i8")
    run_unpacked(wl("cyc", 9, 2, d, ("noise",), "any"))


# ------------------------------------------------------ one-node encoder ----
@pytest.mark.parametrize("code,P,s,d", [("rep", 15, 2, 3001), ("cyc", 15, 2, 3001), ("cyc", 45, 3, 2048), ("cyc", 5, 2, 7), ("cyc", 20, 8, 2051), ("cyc", 21, 10, 1030), ("cyc", 45, 16, 1030)])
def test_encode_node_is_bit_identical_to_the_all_node_form(code, P, s, d):
    w = wl(code, P, s, d)
    c = Case(w)
    try:
        c.encode()
        r = w.r
        for node in range(P):
            rows = [(node // r) * r + t for t in range(r)] if code == "rep" else [(node + t) % P for t in range(r)]
            Gn = c.G[rows].contiguous()
            z = torch.full((c.ld_m,), float("nan"), dtype=torch.float32, device=c.device)
            c.plan.encode_node(node, Gn, z)
            torch.cuda.synchronize()
            assert torch.equal(z[:c.mlen].view(torch.int32), c.Z[node, :c.mlen].view(torch.int32)), node
    finally:
        c.close()


@pytest.mark.parametrize("second", ["f32", "bf16", "i8"])
@pytest.mark.parametrize("P,s,d", [(15, 2, 3001), (45, 3, 2050), (21, 10, 1030), (45, 16, 1031), (40, 17, 515)])
def test_encode_node_on_the_two_word_wires(P, s, d, second):
    """A compute node's own call on its 2s+1 gradients writes both words of its message exactly as
    the all-node encoder does: every window width's kernel against the one-node kernel, bit for bit."""
    c = Case(wl("cyc", P, s, d), wide=second)
    try:
        c.encode()
        torch.cuda.synchronize()
        r = 2 * s + 1
        for node in (0, 1 % P, (P - 2 * s) % P, P - 1):
            Gn = c.G[[(node + t) % P for t in range(r)]].contiguous()
            z = torch.full((c.ld_m,), float("nan"), dtype=torch.float32, device=c.device)
            zl = torch.full((c.ld_m,), 77 if second == "i8" else float("nan"), dtype=c.Zlo.dtype, device=c.device)
            c.plan.encode_node_wide(node, Gn, z, zl)
            torch.cuda.synchronize()
            assert torch.equal(z[:c.mlen].view(torch.int32), c.Z[node, :c.mlen].view(torch.int32)), node
            bits = {"f32": torch.int32, "bf16": torch.int16, "i8": torch.int8}[second]
            assert torch.equal(zl[:c.mlen].view(bits), c.Zlo[node, :c.mlen].view(bits)), node
            assert torch.isnan(z[c.mlen:]).all()
            assert (zl[c.mlen:] == 77).all() if second == "i8" else torch.isnan(zl[c.mlen:].float()).all()
        rep = B.Plan(B.CODE_REPETITION, 15, 2, 100)
        try:
            with pytest.raises(B.DracoError) as e:
                rep.encode_node_wide(0, c.G[:5], c.Z[0], torch.zeros_like(c.Z[0]))
            assert e.value.status == B.EINVAL
        finally:
            rep.close()
    finally:
        c.close()


# ---------------------------------------------------------- random sweep -----
def test_random_shapes_and_attacks():
    """Seeded random (code, P, s, d, adversary count, attack mix, placement) cases."""
    rng = np.random.default_rng(20180309877)
    kinds = ["noise", "signflip", "offset", "constant"]
    for case in range(40):
        code = "rep" if case % 2 == 0 else "cyc"
        s = int(rng.integers(0, 8))
        r = 2 * s + 1
        if code == "rep":
            P = r * int(rng.integers(1, max(2, 60 // r)))
        else:
            P = int(rng.integers(r, 64))
        d = int(rng.integers(1, 30_000))
        a = int(rng.integers(0, s + 1))
        attacks = tuple(rng.choice(kinds, a))
        sigma = float(rng.choice([1.0, 1e-2]))
        w = wl(code, P, s, d, attacks, "any", sigma, seed=100 + case)
        run_and_check(w)


def test_many_small_random_decodes():
    """300 small seeded cases (P < 64, s <= 7, d < 600, 0..s adversaries adding noise of
    0.03 to 1000 times the message scale): both decoder forms against the oracle on the same
    fp32 messages -- status and mask exact, sum within tolerance."""
    rng = np.random.default_rng(11)
    dev = torch.device("cuda:0")
    for case in range(300):
        s = int(rng.integers(1, 8))
        P = int(rng.integers(2 * s + 1, 64))
        d = int(rng.integers(8, 600))
        plan = B.Plan(B.CODE_CYCLIC, P, s, d)
        try:
            mlen = plan.message_len
            ld = synth.padded_len(mlen)
            G = rng.standard_normal((P, d)).astype(np.float32)
            Z = np.zeros((P, ld), dtype=np.float32)
            Z[:, :mlen] = o.encode_cyclic(G, s).astype(np.float32)
            a = int(rng.integers(0, s + 1))
            V = rng.choice(P, a, replace=False)
            mag = 10.0 ** rng.uniform(-1.5, 3)
            scale = np.median(np.abs(Z[:, :mlen]))
            for j in V:
                Z[j, :mlen] += (rng.standard_normal(mlen) * mag * scale).astype(np.float32)
            f = (rng.standard_normal(mlen // 2) + 1).astype(np.float32)
            uo, mo, so = o.decode_cyclic(Z[:, :mlen], f, s, d)
            assert so == o.OK and sorted(np.flatnonzero(mo)) == sorted(V), (case, P, s, d, a, mag)
            R = torch.from_numpy(Z).to(dev)
            fd = torch.from_numpy(f).to(dev)
            u = torch.zeros(synth.padded_len(d), device=dev)
            for fn in (plan.decode_cyclic, plan.decode_cyclic_hostphi):
                m, st = fn(R, fd, u)
                assert st == B.OK and np.array_equal(m, mo), (case, P, s, d, a, mag)
                assert rel_l2(u[:d].cpu().numpy(), uo) <= TOL_SUM["cyc"], (case, P, s, d, a, mag)
        finally:
            plan.close()


def test_many_small_random_votes():
    """300 small seeded repetition cases: 0..s liars per group (sometimes more, then the status
    must say so), edits from one flipped bit in one coordinate to whole-row noise, sometimes
    colluding liars that send the same wrong vector."""
    rng = np.random.default_rng(12)
    dev = torch.device("cuda:0")
    for case in range(300):
        s = int(rng.integers(0, 9))
        r = 2 * s + 1
        P = r * int(rng.integers(1, max(2, 70 // r)))
        d = int(rng.integers(1, 700))
        plan = B.Plan(B.CODE_REPETITION, P, s, d)
        try:
            ld = synth.padded_len(d)
            G = rng.standard_normal((P, d)).astype(np.float32)
            Z = np.zeros((P, ld), dtype=np.float32)
            Z[:, :d] = o.encode_repetition(G, s).astype(np.float32)
            overload = s > 0 and rng.random() < 0.1
            for g in range(P // r):
                a = int(rng.integers(0, s + 1)) if not (overload and g == 0) else s + 1
                liars = g * r + rng.choice(r, a, replace=False)
                shared = rng.standard_normal(d).astype(np.float32)
                collude = rng.random() < 0.3
                for j in liars:
                    kind = int(rng.integers(0, 3))
                    if collude:
                        Z[j, :d] = shared
                    elif kind == 0:
                        Z[j, :d].view(np.uint32)[int(rng.integers(d))] ^= np.uint32(1) << np.uint32(rng.integers(32))
                    elif kind == 1:
                        Z[j, :d] = rng.standard_normal(d).astype(np.float32) * 100
                    else:
                        Z[j, :d] *= np.float32(-100)
                        Z[j, int(rng.integers(d))] += np.float32(1)     # also differs where the message is 0
            uo, mo, so = o.decode_repetition(Z[:, :d], s)
            R = torch.from_numpy(Z).to(dev)
            u = torch.zeros(ld, device=dev)
            m, st = plan.decode_repetition(R, u)
            assert st == so, (case, P, s, d)
            if so == o.OK:
                assert np.array_equal(m, mo), (case, P, s, d)
                got = u[:d].cpu().numpy()
                ok = np.isfinite(uo)
                assert rel_l2(got[ok], uo[ok]) <= TOL_SUM["rep"], (case, P, s, d)
        finally:
            plan.close()


def test_random_shapes_and_attacks_on_the_other_wires():
    """The same kind of sweep for the cyclic code's wide and unpacked wires."""
    rng = np.random.default_rng(1803098770)
    kinds = ["noise", "signflip", "offset"]
    for case in range(24):
        s = int(rng.integers(0, 7))
        P = int(rng.integers(2 * s + 1, 48))
        d = int(rng.integers(1, 20_000))
        a = int(rng.integers(0, s + 1))
        attacks = tuple(rng.choice(kinds, a))
        w = wl("cyc", P, s, d, attacks, "any", float(rng.choice([1.0, 1e-2])), seed=500 + case)
        if case % 4 == 0:
            run_wide(w)
        elif case % 4 == 2:     # these wires' floors depend on (P, s); parity is the check here
            run_wide(w, "bf16" if case % 8 == 2 else "i8", e2e=1e-3)
        else:
            run_unpacked(w, e2e=1.0)          # the fp32-wire floor depends on (P, s); parity is the check here


# ------------------------------------------------- B > P (per-sample rows) ----
@pytest.mark.parametrize("code,P,s,m,d", [
    ("rep", 15, 2, 4, 3001), ("rep", 45, 2, 4, 20_003), ("rep", 9, 1, 16, 999), ("rep", 34, 8, 3, 777),
    ("cyc", 15, 2, 4, 3001), ("cyc", 45, 3, 4, 20_002), ("cyc", 45, 3, 16, 5_001), ("cyc", 15, 7, 2, 2_050),
    ("cyc", 20, 8, 3, 1_001), ("cyc", 6, 0, 5, 4_099), ("cyc", 45, 5, 4, 8_000), ("cyc", 21, 10, 2, 1_030), ("cyc", 25, 12, 2, 515),
    # rows that end next to a piece, a wavefront stride and a window of the workgroup footprint
    ("cyc", 45, 3, 4, 32_769), ("cyc", 9, 1, 4, 8_193), ("rep", 9, 1, 4, 32_767), ("cyc", 9, 1, 8, 65_537), ("cyc", 9, 2, 16, 257),
])
def test_encode_samples_sums_the_unit_gradients_in_the_encoder(code, P, s, m, d):
    """B = m*P per-sample gradients (the paper runs B = 180 and 720 on P = 45): unit gradient k
    is the sum of rows k*m .. k*m+m-1, then the code's encoder."""
    plan = B.Plan(B.CODE_REPETITION if code == "rep" else B.CODE_CYCLIC, P, s, d)
    try:
        ld = synth.padded_len(d)
        S = synth.make_gradients(P * m, d, 1.0, synth.SEED_BASE + 31 * m + P, device="cuda:0", ld=ld)
        mlen = plan.message_len
        Z = torch.full((P, synth.padded_len(mlen)), float("nan"), dtype=torch.float32, device="cuda:0")
        print(f"samples case {code} P={P} s={s} m={m} d={d}", flush=True)
        plan.encode_samples(S, Z)
        torch.cuda.synchronize()
        units = S[:, :d].double().reshape(P, m, d).sum(1).cpu().numpy()
        Zo = o.encode_repetition(units, s) if code == "rep" else o.encode_cyclic(units, s)
        Zg = Z[:, :mlen].cpu().numpy()
        for j in range(P):
            assert rel_l2(Zg[j], Zo[j]) <= 1e-6, j
        if Z.shape[1] > mlen:
            assert torch.isnan(Z[:, mlen:]).all()
        if code == "rep":
            r = 2 * s + 1
            for j in range(P):
                assert np.array_equal(Zg[j].view(np.uint32), Zg[(j // r) * r].view(np.uint32))
        with pytest.raises(B.DracoError):
            plan.encode_samples(S[:P * m - 1], Z)                       # B not a multiple of P
    finally:
        plan.close()


@pytest.mark.parametrize("second", ["f32", "bf16", "i8"])
@pytest.mark.parametrize("P,s,m,d", [(45, 5, 4, 8_002), (15, 2, 8, 3_001), (9, 1, 12, 8_193), (20, 8, 3, 1_001),
                                     (25, 12, 2, 515), (45, 3, 4, 32_769)])
def test_encode_samples_on_the_two_word_wires(P, s, m, d, second):
    """B = m*P sample rows on every two-word wire and through every B > P kernel (four rows per unit,
    rings of eight and four, the general form, the wide-window form): hi + lo against the oracle's
    fp64 message to what the wire carries, element by element, and the second word bit for bit
    wherever the first words agree."""
    plan = B.Plan(B.CODE_CYCLIC, P, s, d)
    try:
        plan.set_second_word({"f32": B.SECOND_WORD_F32, "bf16": B.SECOND_WORD_BF16, "i8": B.SECOND_WORD_I8}[second])
        ld = synth.padded_len(d)
        S = synth.make_gradients(P * m, d, 1.0, synth.SEED_BASE + 37 * m + P, device="cuda:0", ld=ld)
        mlen = plan.message_len
        ldm = synth.padded_len(mlen)
        Z = torch.full((P, ldm), float("nan"), dtype=torch.float32, device="cuda:0")
        lo_dtype = {"f32": torch.float32, "bf16": torch.bfloat16, "i8": torch.int8}[second]
        Zlo = torch.full((P, ldm), 77 if second == "i8" else float("nan"), dtype=lo_dtype, device="cuda:0")
        print(f"wide samples case P={P} s={s} m={m} d={d} second word {second}", flush=True)
        plan.encode_samples_wide(S, Z, Zlo)
        torch.cuda.synchronize()
        units = S[:, :d].double().reshape(P, m, d).sum(1).cpu().numpy()
        Zo = o.encode_cyclic(units, s)
        Zhi = Z[:, :mlen].cpu().numpy()
        Zl = second_word_values(Zhi, Zlo[:, :mlen], second)
        bits = WIDE[second][0]
        for j in range(P):
            slack = 2.0 ** -bits * np.abs(Zo[j]) + 2.0 ** -43 * np.abs(Zo[j]).max()
            assert (np.abs(Zhi[j].astype(np.float64) + Zl[j] - Zo[j]) <= slack).all(), j
        hi_o, lo_o = o.two_word_wire(Zo, second)
        same_hi = Zhi.view(np.uint32) == hi_o.view(np.uint32)
        assert same_hi.mean() >= 0.8
        if second != "f32":
            same_lo = (Zl == lo_o) | (np.abs(Zl - lo_o) <= 2.0 ** -43 * np.abs(Zo).max())
            assert same_lo[same_hi].mean() >= 0.99
        if ldm > mlen:
            assert torch.isnan(Z[:, mlen:]).all()
            assert (Zlo[:, mlen:] == 77).all() if second == "i8" else torch.isnan(Zlo[:, mlen:].float()).all()
    finally:
        plan.close()


# ------------------------------------------------------------ arguments -----
def test_one_shot_forms():
    """The three calls without a plan: encode(assign, grads) -> messages and
    decode(messages, P, s) -> (sum, mask), the plans cached inside the library."""
    dev = torch.device("cuda:0")
    for code, P, s, d in ((B.CODE_REPETITION, 15, 2, 4099), (B.CODE_CYCLIC, 15, 2, 4099), (B.CODE_CYCLIC, 15, 2, 4100)):
        G = synth.make_gradients(P, d, 1.0, 4242, device=dev)
        A = o.assign_repetition(P, s) if code == B.CODE_REPETITION else o.assign_cyclic(P, s)
        Z = B.encode(A, code, G, d)
        Zo = o.encode_repetition(G[:, :d].cpu().numpy(), s) if code == B.CODE_REPETITION else \
            o.encode_cyclic(G[:, :d].cpu().numpy(), s)
        for j in range(P):
            assert_message_close(Z[j].cpu().numpy(), Zo[j], 2 * (2 * s + 1), j)
        R = torch.nn.functional.pad(Z.contiguous(), (0, (-Z.shape[1]) % 4))          # rows 16-byte aligned
        mlen = Z.shape[1]
        R[3, :mlen] = -100.0 * R[3, :mlen]
        ref = G[:, :d].double().sum(0).cpu().numpy()
        for _ in range(2):                                                 # second call reuses the plan
            if code == B.CODE_REPETITION:
                u, mask, status = B.decode_repetition(R[:, :mlen], P, s)
            else:
                u, mask, status = B.decode_cyclic(R[:, :mlen], P, s, d)
            assert status == B.OK and list(np.flatnonzero(mask)) == [3]
            assert u.shape == (d,) and rel_l2(u.cpu().numpy(), ref) <= 1e-5
        # a matrix that is not the code's allocation is refused
        bad = A.copy()
        bad[0, 0], bad[0, (2 * s + 1) % P] = 0, 1
        with pytest.raises(B.DracoError) as e:
            B.encode(bad, code, G, d)
        assert e.value.status == B.EINVAL
    # B > P through the same call: 4 per-sample rows per unit gradient
    P, s, d, m = 9, 1, 1030, 4
    S = synth.make_gradients(P * m, d, 1.0, 77, device=dev)
    Z = B.encode(o.assign_cyclic(P, s), B.CODE_CYCLIC, S, d)
    units = S[:, :d].double().reshape(P, m, d).sum(1).cpu().numpy()
    Zo = o.encode_cyclic(units, s)
    for j in range(P):
        assert_message_close(Z[j].cpu().numpy(), Zo[j], 2, j)
    B.lib().draco_cache_clear()


def test_every_generated_decode_draws_another_projection_vector():
    """f_dev = NULL: a plan's decodes use seed_0 = base, then other seeds; the seed a decode
    used is reported, and the oracle decoding with ITS generator on that seed agrees."""
    w = wl("cyc", 15, 2, 10_007, ("offset", "noise"), "any", 1.0)
    c = Case(w)
    try:
        c.encode()
        c.receive()
        R_host = c.R[:, :c.mlen].cpu().numpy()
        c.plan.set_projection_seed(41)
        seeds = []
        for k in range(3):
            c.u.fill_(float("nan"))
            mask, status = c.plan.decode_cyclic(c.R, None, c.u)
            torch.cuda.synchronize()
            seeds.append(c.plan.last_projection_seed())
            uo, mo, so = o.decode_cyclic(R_host, o.projection_vector(c.mlen // 2, seeds[-1]), w.s, w.d)
            assert status == so == B.OK and np.array_equal(mask, mo) and np.array_equal(mask, c.expected_mask())
            assert_sum_close(c.u[:w.d].cpu().numpy(), uo, TOL_SUM["cyc"], k)
        assert seeds[0] == 41 and len(set(seeds)) == 3
        c.plan.set_projection_seed(41)                     # the same base replays the same sequence
        c.plan.decode_cyclic(c.R, None, c.u)
        assert c.plan.last_projection_seed() == 41
        c.plan.decode_cyclic_hostphi(c.R, None, c.u)
        assert c.plan.last_projection_seed() == seeds[1]
        other = B.Plan(B.CODE_CYCLIC, 15, 2, 10_007)      # two plans start from different bases
        other2 = B.Plan(B.CODE_CYCLIC, 15, 2, 10_007)
        u2 = torch.zeros_like(c.u)
        other.decode_cyclic(c.R, None, u2)
        other2.decode_cyclic(c.R, None, u2)
        assert other.last_projection_seed() != other2.last_projection_seed()
        other.close()
        other2.close()
    finally:
        c.close()


# ------------------------------------------------ the parameter server's update -----
@pytest.mark.parametrize("d", [1, 3, 4, 1023, 1024, 1025, 1_000_003])
def test_apply_update_against_the_oracle(d):
    """params <- params - (lr/B) * sum: one fused multiply-add per parameter in fp32 against
    the oracle's fp64 step; padding beyond d untouched."""
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev)
    g.manual_seed(d)
    n = synth.padded_len(d) + 8
    w0 = torch.randn(n, generator=g, device=dev)
    u = torch.randn(n, generator=g, device=dev) * 30
    lr, Bsz = 0.1, 180
    w = w0.clone()
    B.draco_apply_update(w, u, d, lr / Bsz)
    torch.cuda.synchronize()
    want = o.sgd_update(w0[:d].cpu().numpy(), u[:d].cpu().numpy(), np.float32(lr / Bsz), 1)
    got = w[:d].cpu().numpy().astype(np.float64)
    # one rounding of the fused result: half an ulp of the result
    assert np.all(np.abs(got - want) <= 2.0 ** -24 * (1 + 1e-6) * np.abs(want) + 1e-30)
    assert torch.equal(w[d:], w0[d:])
    B.draco_apply_update(w, u, d, 0.0)
    assert torch.equal(w[:d].cpu(), torch.from_numpy(got.astype(np.float32)))


def test_decode_then_update_is_the_clean_sgd_step():
    """Sec. 2's update fed by D^Rep: with two liars the model after the step is the one
    plain mini-batch SGD reaches on the honest gradients."""
    w = wl("rep", 15, 2, 50_003, ("signflip", "noise"), "distinct_groups")
    c = Case(w)
    try:
        c.encode()
        c.receive()
        mask, status = c.decode()
        assert status == B.OK and np.array_equal(mask, c.expected_mask())
        params = torch.randn(c.u.numel(), device=c.device)
        p0 = params.clone()
        lr = 0.05
        B.draco_apply_update(params, c.u, w.d, lr / w.P)
        torch.cuda.synchronize()
        want = o.sgd_update(p0[:w.d].cpu().numpy(), c.G[:, :w.d].double().sum(0).cpu().numpy(), lr, w.P)
        assert max_abs_err(params[:w.d].cpu().numpy(), want) <= 1e-6 * float(np.max(np.abs(want)))
    finally:
        c.close()


def test_alignment_and_argument_errors():
    w = wl("rep", 6, 1, 100)
    c = Case(w)
    try:
        L = B.lib()
        st = torch.cuda.current_stream().cuda_stream
        assert L.draco_encode(c.plan._h, c.G.data_ptr() + 4, c.ld_g, c.Z.data_ptr(), c.ld_m, st) == B.EALIGN
        assert L.draco_encode(c.plan._h, c.G.data_ptr(), c.ld_g + 1, c.Z.data_ptr(), c.ld_m, st) == B.EALIGN
        assert L.draco_encode(c.plan._h, c.G.data_ptr(), 96, c.Z.data_ptr(), c.ld_m, st) == B.EALIGN
        assert L.draco_encode(c.plan._h, None, c.ld_g, c.Z.data_ptr(), c.ld_m, st) == B.EINVAL
        words = np.zeros(1, dtype=np.uint64)
        assert L.draco_decode_cyclic(c.plan._h, c.Z.data_ptr(), c.ld_m, c.G.data_ptr(), c.u.data_ptr(),
                                     words.ctypes.data, st) == B.EINVAL          # wrong code for the call
    finally:
        c.close()


def test_first_decode_of_a_process_records_its_kernel_alone():
    """In a process of its own: the first decode of (33, 3, 400 001) on one word, whose second kernel locates and recombines, 20 us.
    With the kernel's code brought to the device by that launch the record held 300 to 1700 us; 150 is the bound."""
    code = (
        "import torch\n"
        "from paper_1803_09877_amd import binding as B\n"
        "plan = B.Plan(B.CODE_CYCLIC, 33, 3, 400_001)\n"
        "plan.prepare()\n"
        "plan.set_timing(4)\n"
        "Z = torch.randn((33, 400_004), device='cuda:0')\n"
        "u = torch.zeros(400_004, device='cuda:0')\n"
        "torch.cuda.synchronize()\n"
        "plan.decode_cyclic(Z, None, u)\n"
        "print('us', plan.kernel_times(B.KIND_RECOMBINE)[0] * 1e3)\n")
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    res = subprocess.run([sys.executable, "-c", code], cwd=root, capture_output=True, text=True, timeout=100)
    assert res.returncode == 0, res.stderr[-500:]
    assert float(res.stdout.split("us")[-1]) <= 150.0, res.stdout
