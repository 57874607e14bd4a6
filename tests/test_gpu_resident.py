"""The decode kernel with register-resident weights at the edges of what it holds: the widest and
narrowest layers of every size class and one unit beyond, output layers that just fill the column
tiles, the tail columns and no longer, one and two layers, one utterance, teams whose list is longer
than the rows they decode at a time, more utterances than one launch takes, and label-dense stretches.
Against the oracle, through the C ABI.  Also its gates alone, and what engines do between the two
kernels: refused configurations and allocations, launches on request, threads."""
import dataclasses

import numpy as np
import pytest

import oracle
import synth
from parity_util import compare
from test_gpu_parity import N_THREADS, check, pkg, run_gpu  # noqa: F401  (pkg: fixture)

pytestmark = pytest.mark.gpu


def model_inputs(H, J, V1, L, B, T, seed, durations=(), big_blanks=(), max_symbols=4, F=32):
    dims = synth.ModelDims(F=F, E=24, H=H, L=L, J=J, V1=V1, durations=tuple(durations), big_blanks=tuple(big_blanks))
    model = synth.make_model(dims, seed, weight_range=0.15, emb_gain=4.0, pred_gain=3.0, blank_bias=1.5)
    x, ln = synth.make_inputs(seed, B, T, dims.F, 0, T)
    variant = "tdt" if durations else "label"
    return synth.Workload(f"resident {H}/{J}/{V1}/{L}", variant, model, x, ln, max_symbols)


# (H, J, V1, L): widths of the size classes 128, 320 and 640 and their neighbours; output layers of
# 32 columns per work-group (8, 16, 32 of them), with a full tail, and one more
EDGES = [(4, 4, 3, 1), (128, 128, 256, 1), (132, 128, 257, 2), (128, 132, 264, 1), (320, 316, 512, 2), (316, 320, 528, 1),
         (324, 320, 529, 1), (640, 640, 1024, 1), (640, 636, 1056, 2), (636, 640, 1057, 1), (644, 640, 40, 1), (160, 640, 33, 2)]


@pytest.mark.parametrize("H,J,V1,L", EDGES)
@pytest.mark.parametrize("bf16", [False, True])
def test_edges_of_the_size_classes(pkg, H, J, V1, L, bf16):  # noqa: F811
    w = model_inputs(H, J, V1, L, B=9, T=14, seed=H + J + V1)
    eng = pkg.Engine(w.model, w.B, w.T, flags=pkg.RNNT_FLAG_BF16_ARITHMETIC if bf16 else 0)
    for variant in ("label", "frame"):
        check(pkg, w, variant, f"edge {H}/{J}/{V1}/{L} bf16={bf16}", engine=eng, bf16=bf16, logp=True)
    one = dataclasses.replace(w, enc_out=w.enc_out[:1].copy(), enc_len=np.maximum(w.enc_len[:1], 3))
    check(pkg, one, "label", f"edge {H}/{J}/{V1}/{L} bf16={bf16}, one utterance", engine=eng, bf16=bf16)
    eng.close()


@pytest.mark.parametrize("B", [2, 33, 70, 773])
@pytest.mark.parametrize("extra", [{}, dict(durations=(0, 1, 3, 7)), dict(big_blanks=(2, 5))])
def test_lists_longer_than_the_rows_in_work(pkg, B, extra):  # noqa: F811
    """Every decoder with one row per team, a partly filled last row, rows that take over the next
    utterance of the team's list, and (773 utterances on 6 teams that take 128 each) a second launch."""
    w = model_inputs(324, 332, 530 if not extra else 520, 2, B=B, T=9, seed=B, **extra)
    eng = pkg.Engine(w.model, w.B, w.T)
    check(pkg, w, w.variant, f"list {B} {extra}", engine=eng, logp=True)
    eng.close()


def test_two_threads_on_streams_of_their_own(pkg):  # noqa: F811
    """Decodes of two engines from two threads at once: their work-groups may not share the device."""
    import threading

    import torch
    jobs = []
    for seed, B in ((3, 1), (4, 40)):
        w = model_inputs(324, 332, 530, 2, B=B, T=40, seed=seed)
        eng = pkg.Engine(w.model, w.B, w.T)
        enc, ln = torch.from_numpy(w.enc_out).cuda(), torch.from_numpy(w.enc_len.astype(np.int32)).cuda()
        want = eng.decode("label", enc, ln, w.max_symbols)["tokens"].clone()
        jobs.append((eng, enc, ln, w.max_symbols, want, []))
    torch.cuda.synchronize()

    def work(eng, enc, ln, S, want, same):
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            for _ in range(20):
                out = eng.decode("label", enc, ln, S)
                stream.synchronize()
                same.append(bool(torch.equal(out["tokens"], want)))

    threads = [threading.Thread(target=work, args=j) for j in jobs]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for eng, _, _, _, _, same in jobs:
        assert eng.status() == 0 and same == [True] * 20
        eng.close()


def test_cooperative_launches_on_request(pkg):  # noqa: F811
    """Engines of either kernel that launch cooperatively, beside one that does not."""
    for L in (1, 2, 3):
        w = model_inputs(324, 332, 530, L, B=33, T=12, seed=50 + L)
        coop = pkg.Engine(w.model, w.B, w.T, flags=pkg.RNNT_FLAG_COOPERATIVE_LAUNCH)
        plain = pkg.Engine(w.model, w.B, w.T)
        for v in ("label", "frame", "label_noalloc"):
            check(pkg, w, v, f"cooperative {L}", engine=coop)
            check(pkg, w, v, f"ordinary {L}", engine=plain)
        coop.close()
        plain.close()


@pytest.mark.parametrize("L", [2, 3])
def test_a_refused_configuration_changes_nothing(pkg, L):  # noqa: F811
    """A fresh engine, and one with a layout and a lookahead of its own, decode after a refused
    rnnt_engine_configure (teams that do not divide the device, joint groups that do not divide a
    team, more than 16 utterances per team) with what was in force before it."""
    w = model_inputs(324, 332, 530, L, B=40, T=12, seed=40 + L)
    refused = [dict(n_teams=3), dict(n_teams=8, joint_groups=3), dict(n_teams=2), dict(joint_groups=2), dict(lookahead=33),
               dict(n_teams=7, lookahead=4), dict(n_teams=3, search_steps=2), dict(search_steps=-2)]
    eng = pkg.Engine(w.model, w.B, w.T)
    for knobs in ({}, dict(n_teams=8, joint_groups=2, lookahead=3, search_steps=2), dict(lookahead=5)):
        eng.configure(**knobs)
        in_force = ("n_teams", "team_size", "joint_groups", "lookahead", "search_steps")
        before = {v: check(pkg, w, v, f"in force {knobs}", engine=eng)[2] for v in ("label", "frame", "label_noalloc")}
        for bad in refused:
            with pytest.raises(pkg.RnntError) as err:
                eng.configure(**bad)
            assert err.value.code == -2, bad
            for v in ("label", "frame", "label_noalloc"):
                after = check(pkg, w, v, f"refused {bad}", engine=eng)[2]
                assert [after[k] for k in in_force] == [before[v][k] for k in in_force], (knobs, bad, v)
    eng.close()


def test_the_default_lookahead_after_a_return_to_the_resident_kernel(pkg):  # noqa: F811
    """Layouts sized for another lookahead are replanned when the streaming kernel is asked for again:
    96 utterances of a TDT model in three rows per joint group, 8 frames each, not the 5 that fit
    layouts made for one."""
    w = model_inputs(324, 332, 520, 2, B=96, T=12, seed=96, durations=(0, 1, 3))
    eng = pkg.Engine(w.model, w.B, w.T)
    for knobs, lookahead in ((dict(lookahead=1), 1), (dict(), None), (dict(search_steps=1), 8)):
        eng.configure(**knobs)
        stats = check(pkg, w, "tdt", f"lookahead after {knobs}", engine=eng)[2]
        if lookahead is not None:
            assert stats["lookahead"] == lookahead and stats["n_teams"] == 16
    eng.close()


@pytest.mark.parametrize("is_tanh", [False, True])
def test_gates_pass_on_nan_and_saturate_at_infinity(pkg, is_tanh):  # noqa: F811
    x = np.array([np.nan, -np.nan, np.inf, -np.inf, 1e30, -1e30, 0.0, -0.0], dtype=np.float32)
    got = pkg.rnnt_probe_gate(is_tanh, x)
    assert np.isnan(got[:2]).all()
    if is_tanh:
        assert got[2:].tolist() == [1.0, -1.0, 1.0, -1.0, 0.0, 0.0]
    else:
        assert got[2] == got[4] == 1.0 and got[6] == got[7] == 0.5
        assert 0.0 <= got[3] <= 2e-38 and 0.0 <= got[5] <= 2e-38          # exp(-87), where the argument is limited


@pytest.mark.parametrize("is_tanh,ulps", [(False, 2.6), (True, 1.3)])
def test_gates_against_64_bits(pkg, is_tanh, ulps):  # noqa: F811
    """Every 31st float of magnitude 2^-33 to 87, both signs, and zero: within the bound that holds for all of them
    (2.58 and 1.21 units in the last place, measured once over every float), and the sigmoid within 2e-38
    below -87, where its argument is limited."""
    top = int(np.float32(87.0).view(np.uint32))
    bits = np.concatenate([np.arange(0x2F000000, top, 31, dtype=np.uint32), np.array([0, top], dtype=np.uint32)])
    worst = 0.0
    for part in np.array_split(np.concatenate([bits, bits | np.uint32(1 << 31)]), 8):
        x = part.view(np.float32)
        got, xd = pkg.rnnt_probe_gate(is_tanh, x).astype(np.float64), x.astype(np.float64)
        want = np.tanh(xd) if is_tanh else 1.0 / (1.0 + np.exp(-xd))
        ulp = np.ldexp(1.0, np.maximum(np.frexp(want)[1], -125) - 24)
        worst = max(worst, float((np.abs(got - want) / ulp).max()))
    assert worst <= ulps, worst
    if not is_tanh:
        low = np.linspace(-200.0, -87.0, 4096, dtype=np.float32)
        assert np.abs(pkg.rnnt_probe_gate(False, low).astype(np.float64) - 1.0 / (1.0 + np.exp(-low.astype(np.float64)))).max() <= 2e-38


@pytest.mark.parametrize("B", [15, 20])
@pytest.mark.parametrize("extra", [{}, dict(durations=(0, 1)), dict(big_blanks=(2, 5))])
def test_label_dense_and_sparse_stretches(pkg, B, extra):  # noqa: F811
    """Rows of 25 frames with up to four labels each, then 25 blank ones, at different times: teams of three and
    four rows change to half the frames per row and back."""
    dims = synth.ModelDims(F=336, E=24, H=324, L=2, J=332, V1=530, durations=extra.get("durations", ()),
                           big_blanks=extra.get("big_blanks", ()))
    model = synth.make_model(dims, B, weight_range=0.15, emb_gain=4.0, pred_gain=3.0, blank_bias=-1.0)
    # a frame that drives the blank's logit up, whatever the prediction side adds
    want = 60.0 * np.maximum(model.w_out[dims.blank].astype(np.float64), 0.0) - model.b_enc
    blank = np.linalg.lstsq(model.w_enc.astype(np.float64), want, rcond=None)[0].astype(np.float32)
    x, ln = synth.make_inputs(B, B, 100, dims.F, 50, 100)
    t, b = np.arange(100)[None, :], np.arange(B)[:, None]
    x = np.where(((t + 5 * b) // 25 % 2 == 0)[:, :, None], x, blank[None, None]).astype(np.float32)
    w = synth.Workload("dense and sparse", "tdt" if dims.D else "label", model, x, ln, 4)
    eng = pkg.Engine(w.model, w.B, w.T)
    ref, got, stats = check(pkg, w, w.variant, f"dense and sparse {B} {extra}", engine=eng, logp=True)
    import torch
    enc, lens = torch.from_numpy(w.enc_out).cuda(), torch.from_numpy(w.enc_len.astype(np.int32)).cuda()
    for i in range(50):        # the same hand-overs in whatever order they come
        again = eng.decode(w.variant, enc, lens, w.max_symbols, logp=i % 2 == 0)["tokens"].cpu().numpy()
        assert np.array_equal(again, got["raw_tokens"]), i
    assert eng.status() == 0
    eng.close()
    # what a team that never changes examines: `la` frames of every row at every step, as far as it has them
    la, full = stats["lookahead"], 0
    for i in range(B):
        at, n, k, frames, length = 0, 0, 0, ref.frames[i], int(ln[i])
        while at < length:
            full += min(la, length - at)
            if k == len(frames) or frames[k] >= at + la:
                at, n = at + la, 0
                continue
            n = n if frames[k] == at else 0
            at, n, move = int(frames[k]), n + 1, int(ref.durs[i][k])
            if move > 0 or n == w.max_symbols:
                at, n = at + max(move, 1), 0
            k += 1
    print(f"samples {stats['joint_samples']}, without changes {full}", flush=True)
    assert stats["joint_samples"] < 0.95 * full


@pytest.mark.parametrize("extra", [{}, dict(durations=(0, 1, 9, 40)), dict(big_blanks=(2, 33))])
@pytest.mark.parametrize("H,J,V1,L", [(64, 68, 60, 1), (316, 320, 500, 1), (324, 332, 520, 2)])
@pytest.mark.parametrize("bf16", [False, True])
def test_rows_that_end_one_after_the_other(pkg, H, J, V1, L, extra, bf16):  # noqa: F811
    """Four rows a team that end at different times, so that the joint step goes from 8 frames a row to 10, 16 and 31, and
    (two rows a team) from 8 to 16: labels in the first and the last frame that such a step holds, skips beyond it,
    one frame more than the last rows' steps hold, and utterances that start when others have ended."""
    n_teams = {60: 32, 500: 16, 520: 6 if not bf16 else 8}[V1]
    for rows, more in ((4, 2), (2, 0)):
        B = rows * n_teams + more
        w = model_inputs(H, J, V1, L, B=B, T=97, seed=H + rows, F=(J + 15) // 16 * 16, **extra)
        # few labels: a frame without one for most of the frames
        want = 60.0 * np.maximum(w.model.w_out[w.model.dims.blank].astype(np.float64), 0.0) - w.model.b_enc
        blank = np.linalg.lstsq(w.model.w_enc.astype(np.float64), want, rcond=None)[0].astype(np.float32)
        g = np.random.default_rng(B)
        gap = np.array([1, 8, 10, 11, 16, 17, 31, 32, 63])[g.integers(0, 9, (B, 97))].cumsum(1)
        label = (gap[:, :, None] == np.arange(97)[None, None, :] + 1).any(1)
        x = np.where(label[:, :, None], w.enc_out, blank[None, None]).astype(np.float32)
        length = np.sort(g.integers(1, 98, B))[::-1].astype(np.int32)
        length[-more or B:] = 5
        w = dataclasses.replace(w, enc_out=x, enc_len=length)
        eng = pkg.Engine(w.model, w.B, w.T, flags=pkg.RNNT_FLAG_BF16_ARITHMETIC if bf16 else 0)
        check(pkg, w, w.variant, f"rows that end {H}/{J}/{V1}/{L} {extra} {rows} bf16={bf16}", engine=eng, bf16=bf16, logp=not bf16)
        eng.close()


@pytest.mark.parametrize("H,J,V1,L,bf16", [(64, 64, 40, 1, False), (128, 124, 100, 1, False), (100, 128, 255, 1, True), (128, 128, 254, 2, False),
                                           (320, 316, 257, 1, False), (324, 332, 520, 2, False), (324, 332, 520, 2, True)])
@pytest.mark.parametrize("durations", [(2,), (2, 1), (0, 3, 1), (1, 0, 2, 3, 4, 5, 6, 7)])
def test_durations_that_are_no_numbers(pkg, H, J, V1, L, bf16, durations):  # noqa: F811
    """Where every duration's output is NaN the first one is taken, as where all are equal, whatever their number and the model's size."""
    w = model_inputs(H, J, V1, L, B=19, T=23, seed=len(durations), durations=durations)
    nan = np.full(len(durations), np.nan, dtype=np.float32)
    w.model.w_out[V1:], w.model.b_out[V1:] = 0.0, nan
    w.model.b_out[w.model.dims.blank] -= 1.5          # (labels and blanks)
    eng = pkg.Engine(w.model, w.B, w.T, flags=pkg.RNNT_FLAG_BF16_ARITHMETIC if bf16 else 0)
    w.model.b_out[V1:] = 0.0
    _, got, _ = check(pkg, w, "tdt", f"NaN durations {H}/{L}/{bf16} {durations}", engine=eng, bf16=bf16)
    durs = np.concatenate(got["durs"])           # (in the bfloat16 mode another one would pass for a tie)
    assert len(durs) > w.B and (durs == durations[0]).all()
    eng.close()


@pytest.mark.parametrize("H,J,V1,L", [(64, 64, 40, 1), (128, 124, 100, 1), (320, 316, 257, 1), (324, 332, 520, 2)])
@pytest.mark.parametrize("extra", [dict(durations=(0, 2**31 - 1, 1, 2)), dict(durations=(1, 2, 3, 2**31 - 20)), dict(big_blanks=(2, 2**31 - 1))])
@pytest.mark.parametrize("streaming", [False, True])
def test_durations_beyond_any_utterance(pkg, H, J, V1, L, extra, streaming):  # noqa: F811
    """Durations and spans up to the largest int end an utterance from any frame, as 2^30 does, and are reported as they are."""
    w = model_inputs(H, J, V1, L, B=21, T=29, seed=H + 1, **extra)
    w.model.b_out[w.model.dims.blank] -= 0.7
    eng = pkg.Engine(w.model, w.B, w.T)
    if streaming:
        eng.configure(search_steps=2)
    short = lambda v: tuple(min(d, 2**30) for d in v)  # noqa: E731
    dims = dataclasses.replace(w.model.dims, durations=short(w.model.dims.durations), big_blanks=short(w.model.dims.big_blanks))
    near = dataclasses.replace(w, model=dataclasses.replace(w.model, dims=dims, durations=np.minimum(w.model.durations, 2**30)))
    net = oracle.LstmNet(near.model)
    ref = oracle.decode(net, w.enc_out, w.enc_len, w.max_symbols, "seq", n_threads=N_THREADS)
    got, status, _ = run_gpu(eng, w, w.variant, w.max_symbols)
    assert status == 0 and ref.tok_len.sum() > w.B // 2
    assert set(np.concatenate(got["durs"])) <= set(w.model.dims.durations or (0,))
    got["durs"] = [np.minimum(d, 2**30) for d in got["durs"]]
    assert not compare(near, net, ref, got, w.max_symbols)
    eng.close()


def test_an_engine_that_does_not_fit_the_memory_leaves_the_others_alone(pkg):  # noqa: F811
    """The projected frames of 2^27 padded frames take 320 GiB: refused by the allocator, and the next call of an
    engine that exists does not report that error."""
    w = model_inputs(324, 640, 530, 2, B=9, T=12, seed=9)
    eng = pkg.Engine(w.model, w.B, w.T)
    for v in ("label", "frame"):
        with pytest.raises(pkg.RnntError) as err:
            pkg.Engine(w.model, 1 << 14, 1 << 13)
        assert err.value.code == -4
        check(pkg, w, v, "after a refused allocation", engine=eng)
    eng.close()


@pytest.mark.parametrize("extra", [{}, dict(durations=(0, 1, 3, 7)), dict(big_blanks=(2, 5))])
@pytest.mark.parametrize("L,teams", [(1, 8), (2, 6)])
def test_more_utterances_than_one_launch_takes(pkg, L, teams, extra):  # noqa: F811
    """A team takes 128 utterances a launch: three launches, the last of seven utterances, with every output of a
    decoder, and an utterance of large values in the second and third."""
    w = model_inputs(324, 332, 530 if not extra else 520, L, B=2 * teams * 128 + 7, T=5, seed=11, **extra)
    x = w.enc_out.copy()
    x[teams * 128 + 3] *= np.float32(1e6)
    x[2 * teams * 128 + 2] *= np.float32(1e6)
    w = dataclasses.replace(w, enc_out=x)
    eng = pkg.Engine(w.model, w.B, w.T)
    check(pkg, w, w.variant, f"three launches {L} {extra}", engine=eng, logp=True)
    eng.close()


@pytest.mark.parametrize("H,J,V1,L,bf16,teams", [(320, 320, 257, 1, False, 16), (128, 128, 127, 1, False, 32), (128, 128, 127, 2, True, 32)])
def test_full_lists_of_the_smaller_classes(pkg, H, J, V1, L, bf16, teams):  # noqa: F811
    """As many utterances as a launch takes, their lengths ranked in the place of the frames, and seven in another; many of
    the lengths are equal, some are 0."""
    w = model_inputs(H, J, V1, L, B=teams * 128 + 7, T=4, seed=12)
    lens = np.random.default_rng(12).integers(0, 5, w.B).astype(np.int32)
    w = dataclasses.replace(w, enc_len=lens)
    eng = pkg.Engine(w.model, w.B, w.T, flags=pkg.RNNT_FLAG_BF16_ARITHMETIC if bf16 else 0)
    check(pkg, w, w.variant, f"full lists {H} {L}", engine=eng, bf16=bf16)
    eng.close()


@pytest.mark.parametrize("H,J,V1,L", [(128, 128, 255, 1), (316, 320, 529, 1), (324, 640, 530, 2), (640, 636, 1025, 2)])
def test_rows_of_very_different_magnitude(pkg, H, J, V1, L):  # noqa: F811
    """fp32 weights are held as fp16 parts after a power of two for each row: matrices whose rows span 2^-40 to 2^12,
    projected frames of up to 2^12, and a row of zeros.  To the usual bar: a power of two changes no rounding."""
    w = model_inputs(H, J, V1, L, B=5, T=12, seed=H + V1)
    m, rng = w.model, np.random.default_rng(7)

    def scale(n, lo, hi):
        return np.exp2(rng.integers(lo, hi + 1, n)).astype(np.float32)[:, None]

    for a in (m.w_hh[0], m.w_hh[-1], m.w_ih[-1]):
        a *= scale(a.shape[0], -40, 1)
    m.w_pred *= scale(J, -40, 6)
    m.w_enc *= scale(J, -20, 12)
    m.w_out *= scale(m.w_out.shape[0], -40, -10)
    m.w_hh[0][3], m.w_pred[1], m.w_out[2] = 0.0, 0.0, 0.0
    eng = pkg.Engine(m, w.B, w.T)
    check(pkg, w, "label", f"magnitudes {H}/{J}/{V1}/{L}", engine=eng, logp=True)
    eng.close()


def tokens_as_the_oracle_has_them(pkg, w):  # noqa: F811
    """Labels alone, where logits are infinite."""
    import torch

    import oracle
    eng = pkg.Engine(w.model, w.B, w.T)
    out = eng.decode(w.variant, torch.from_numpy(w.enc_out).cuda(), torch.from_numpy(w.enc_len.astype(np.int32)).cuda(), w.max_symbols)
    got, n = out["tokens"].cpu().numpy().reshape(w.B, -1), out["tok_len"].cpu().numpy()
    assert eng.status() == 0
    eng.close()
    ref = oracle.decode(oracle.LstmNet(w.model), w.enc_out, w.enc_len, w.max_symbols, "seq")
    assert n.tolist() == ref.tok_len.tolist()
    for b in range(w.B):
        assert got[b, :n[b]].tolist() == ref.tokens[b].tolist(), b


@pytest.mark.parametrize("value", [np.inf, 3e38])
@pytest.mark.parametrize("H,J,V1,L", [(100, 128, 255, 1), (324, 332, 529, 1), (324, 640, 530, 2)])
def test_projected_frames_without_a_bound(pkg, H, J, V1, L, value):  # noqa: F811
    """One column of the projected frames is infinite, or as large as fp32 holds: the label is the first with an
    infinite logit, or the one with the largest weight, as for the oracle."""
    w = model_inputs(H, J, V1, L, B=20, T=4, seed=H + V1, max_symbols=2)
    m = w.model
    m.b_enc[7] = value
    m.w_out[:9, 7] = -np.abs(m.w_out[:9, 7])         # (not the first label)
    tokens_as_the_oracle_has_them(pkg, w)


def test_weights_that_are_not_finite_run_in_the_streaming_kernel(pkg):  # noqa: F811
    """fp16 parts of an infinite weight do not exist; the bfloat16 mode has none to form."""
    w = model_inputs(324, 332, 530, 2, B=9, T=8, seed=13)
    w.model.w_pred[5, 7] = np.inf
    for flags, streaming in ((0, True), (pkg.RNNT_FLAG_BF16_ARITHMETIC, False)):
        eng = pkg.Engine(w.model, w.B, w.T, flags=flags)
        import torch
        eng.decode("label", torch.from_numpy(w.enc_out).cuda(), torch.from_numpy(w.enc_len.astype(np.int32)).cuda(), w.max_symbols)
        assert eng.status() == 0 and (eng.stats()["search_steps"] != 1) == streaming
        eng.close()


# one layer in the two wider size classes, the widest with a tail column, and two layers
WIDE = [(316, 320, 520, 1), (640, 640, 1025, 1), (324, 640, 530, 2)]


@pytest.mark.parametrize("H,J,V1,L", WIDE)
def test_prediction_biases_that_switch_joint_units_off(pkg, H, J, V1, L):  # noqa: F811
    """-inf and -1e30 of b_pred are zeros behind the relu, and nothing to the other units."""
    w = model_inputs(H, J, V1, L, B=9, T=12, seed=H + 1)
    w.model.b_pred[7], w.model.b_pred[11], w.model.b_pred[J - 1] = -np.inf, -1e30, -3e38
    eng = pkg.Engine(w.model, w.B, w.T)
    check(pkg, w, "label", f"units off {H}/{J}/{V1}/{L}", engine=eng, logp=True)
    eng.close()


@pytest.mark.parametrize("H,J,V1,L", WIDE)
@pytest.mark.parametrize("B", [6, 40])
def test_a_large_utterance_leaves_the_others_alone(pkg, H, J, V1, L, B):  # noqa: F811
    """Utterances of 1e12 and of 3e38 among ordinary ones, and one of 1e-12: every one as the oracle has it."""
    w = model_inputs(H, J, V1, L, B=B, T=10, seed=H + B)
    x = w.enc_out.copy()
    x[1] *= np.float32(1e12)
    x[4] = 0.0
    x[4, :, 0] = 3e38                     # (its projected frames: up to 4.5e37)
    x[5] *= np.float32(1e-12)
    w = dataclasses.replace(w, enc_out=x, enc_len=np.maximum(w.enc_len, 3))
    eng = pkg.Engine(w.model, w.B, w.T)
    check(pkg, w, "label", f"large utterance {H}/{J}/{V1}/{L} {B}", engine=eng, logp=B <= 6)
    eng.close()


@pytest.mark.parametrize("value", [np.inf, 3e38])
@pytest.mark.parametrize("L,durations", [(1, ()), (2, ()), (1, (0, 1, 2, 3, 4)), (2, (0, 1, 2, 3, 4))])
def test_projected_frames_without_a_bound_reach_the_tail_column(pkg, L, durations, value):  # noqa: F811
    """640/640/1025: blank is a tail column, and so are all five durations.  An infinite column of the projected frames
    makes the blank (TDT: label 9 and duration 3) the only infinite output that is positive."""
    V1 = 1025
    w = model_inputs(640, 640, V1, L, B=20, T=6, seed=L, durations=durations, max_symbols=2)
    m = w.model
    m.b_enc[7] = value
    m.w_out[:, 7] = -np.abs(m.w_out[:, 7]) - np.float32(1e-3)
    for row in (9, V1 + 3) if durations else (V1 - 1,):
        m.w_out[row, 7] = 0.125
    tokens_as_the_oracle_has_them(pkg, w)


@pytest.mark.parametrize("value", [np.inf, 3.4e38, 1e30])
@pytest.mark.parametrize("H,J,V1,L", [(100, 128, 255, 1), (324, 332, 529, 1), (324, 640, 530, 2), (640, 640, 1025, 1)])
def test_prediction_biases_without_a_bound(pkg, H, J, V1, L, value):  # noqa: F811
    """A joint unit that its bias makes infinite, or as large as fp32 holds: as for infinite projected frames."""
    w = model_inputs(H, J, V1, L, B=20, T=4, seed=H + V1, max_symbols=2)
    w.model.b_pred[7] = value
    w.model.w_out[:9, 7] = -np.abs(w.model.w_out[:9, 7])         # (not the first label)
    tokens_as_the_oracle_has_them(pkg, w)


# ... and TDT with every duration in the tail
WIDE_TDT = [(*s, ()) for s in WIDE] + [(640, 640, 1025, 1, (0, 1, 2, 3, 4)), (640, 640, 1024, 2, (0, 1, 2, 3, 4))]


@pytest.mark.parametrize("H,J,V1,L,durations", WIDE_TDT)
@pytest.mark.parametrize("B,size", [(3, 1e12), (40, 1e12), (9, 1e30), (9, 1e7)])
def test_a_large_frame_leaves_its_neighbours_alone(pkg, H, J, V1, L, durations, B, size):  # noqa: F811
    """One or two frames of every other utterance are far larger than the rest: every frame as the oracle has it."""
    w = model_inputs(H, J, V1, L, B=B, T=12, seed=H + B, durations=durations)
    x = w.enc_out.copy()
    x[::2, 2] *= np.float32(size)
    x[::4, 7] *= np.float32(size)
    w = dataclasses.replace(w, enc_out=x, enc_len=np.maximum(w.enc_len, 5))
    eng = pkg.Engine(w.model, w.B, w.T)
    check(pkg, w, w.variant, f"large frame {H}/{J}/{V1}/{L} {durations} {B} {size}", engine=eng, logp=B <= 9)
    eng.close()


@pytest.mark.parametrize("H,J,V1,L,durations", WIDE_TDT)
def test_a_joint_unit_with_large_weights_that_is_off(pkg, H, J, V1, L, durations):  # noqa: F811
    """A row of w_pred of 1e9 whose bias of -1e11 its hidden values hardly ever make good: what the unit could be
    says nothing of the others' size."""
    w = model_inputs(H, J, V1, L, B=9, T=12, seed=H + 2, durations=durations)
    w.model.w_pred[5] *= np.float32(1e10 / 0.45)
    w.model.b_pred[5] = -5e11
    eng = pkg.Engine(w.model, w.B, w.T)
    check(pkg, w, w.variant, f"unit off {H}/{J}/{V1}/{L} {durations}", engine=eng, logp=True)
    eng.close()


@pytest.mark.parametrize("L", [1, 2])
@pytest.mark.parametrize("bf16", [False, True])
def test_the_largest_instances(pkg, L, bf16):  # noqa: F811
    """The widest layers with a tail column and two tiles of samples: what takes the most of the LDS."""
    w = model_inputs(640, 640, 1025, L, B=24, T=9, seed=L)
    eng = pkg.Engine(w.model, w.B, w.T, flags=pkg.RNNT_FLAG_BF16_ARITHMETIC if bf16 else 0)
    check(pkg, w, "label", f"largest {L} bf16={bf16}", engine=eng, bf16=bf16, logp=True)
    eng.close()


@pytest.mark.parametrize("J,B,T,durations", [(640, 27, 500, ()), (404, 41, 510, (0, 1, 3, 7))])
def test_large_batches_whose_frames_are_asked_for_ahead(pkg, J, B, T, durations):  # noqa: F811
    """Projected frames of more than 32 MB, the last utterance up to the last row of them, the others short: results with the loads
    ahead (host_pack_check.cpp has which rows they are of)."""
    assert B * T * J * 4 > 32 << 20
    w = model_inputs(324, J, 530, 2, B=B, T=T, seed=J, durations=durations)
    ln = np.minimum(w.enc_len, 17)
    ln[-1], ln[0] = T, T - 3
    w = dataclasses.replace(w, enc_len=ln)
    eng = pkg.Engine(w.model, w.B, w.T)
    check(pkg, w, w.variant, f"ahead {J} {B} {T} {durations}", engine=eng)
    eng.close()


@pytest.mark.parametrize("H,J,V1,L,durations", WIDE_TDT)
@pytest.mark.parametrize("size", [1e7, 1e12])
def test_a_large_joint_unit_that_nobody_reads(pkg, H, J, V1, L, durations, size):  # noqa: F811
    """One unit of every frame is far larger than the others and has no weights in the output layer."""
    w = model_inputs(H, J, V1, L, B=9, T=12, seed=H + 3, durations=durations)
    w.model.b_enc[7] = size
    w.model.w_out[:, 7] = 0.0
    eng = pkg.Engine(w.model, w.B, w.T)
    check(pkg, w, w.variant, f"large unit {H}/{J}/{V1}/{L} {durations} {size}", engine=eng, logp=True)
    eng.close()


# output layers with a tail of one column, of more columns than there are pairs of work-groups, and of one for each of them; teams of
# the three size classes
TAILS = [(128, 128, 257, 1, 32, ()), (128, 128, 264, 1, 32, ()), (124, 128, 254, 1, 32, (0, 1, 2, 3)), (320, 316, 521, 1, 16, ()),
         (320, 316, 528, 1, 16, ()), (640, 636, 1026, 2, 6, ()), (640, 636, 1056, 2, 6, ()), (640, 640, 1048, 1, 8, (0, 1, 2, 0, 3, 1, 2, 4))]


@pytest.mark.parametrize("H,J,V1,L,teams,durations", TAILS)
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("dense", [False, True])
def test_tails_of_steps_with_two_tiles(pkg, H, J, V1, L, teams, durations, bf16, dense):  # noqa: F811
    """Three and four rows a team, whose joint steps are shared out over pairs of work-groups: tail columns of either one, equal ones (the
    lowest index wins), durations among them, and (dense: four labels on every frame) steps of one tile in between."""
    w = model_inputs(H, J, V1, L, B=3 * (teams if L == 1 or not bf16 else 8) + 2, T=14, seed=H + V1, durations=durations)
    m, first = w.model, V1 + len(durations) - len(range((V1 + len(durations)) % (32 * {640: 32, 320: 16, 128: 8, 124: 8}[H])))
    same = [first, first + 3, first + 5] if first + 5 < V1 - 1 else []
    for i in same[1:]:
        m.w_out[i], m.b_out[i] = m.w_out[same[0]], m.b_out[same[0]]
    if same:
        m.b_out[same] += np.float32(3.0)          # (labels of the tail are found now and then)
    if dense:
        m.b_out[m.dims.blank] -= np.float32(4.0)
    eng = pkg.Engine(m, w.B, w.T, flags=pkg.RNNT_FLAG_BF16_ARITHMETIC if bf16 else 0)
    _, got, _ = check(pkg, w, w.variant, f"tails {H}/{J}/{V1}/{L} {durations} bf16={bf16} dense={dense}", engine=eng, bf16=bf16, logp=not bf16)
    labels = np.concatenate(got["tokens"])
    assert not same or ((labels == same[0]).any() and not np.isin(labels, same[1:]).any())
    eng.close()


# (bfloat16 mode: no layers of 640.  Its margin, 2e-2, is about twice what a step of bfloat16, 2^-8 of a value, makes of logits of up to 3
# at a time; those of 332 reach 9 with these inputs, those of 640 reach 19.)  Every kind and precision in every size class.
EIGHT = [(64, 68, 60, 1, False, 32), (128, 128, 257, 2, True, 32), (316, 320, 529, 1, False, 8), (320, 316, 500, 1, True, 16),
         (100, 128, 250, 2, False, 24), (324, 332, 1040, 2, False, 6), (324, 332, 1040, 2, True, 8), (640, 636, 1025, 1, False, 8),
         (324, 332, 1040, 1, True, 8), (128, 124, 257, 1, True, 32), (320, 316, 500, 2, True, 16), (316, 320, 500, 2, False, 12)]


@pytest.mark.parametrize("H,J,V1,L,bf16,teams", EIGHT)
@pytest.mark.parametrize("extra", [{}, dict(durations=(0, 1, 3, 9)), dict(big_blanks=(2, 7))])
@pytest.mark.parametrize("more", [0, 3])
def test_eight_rows_a_team(pkg, H, J, V1, L, bf16, teams, extra, more):  # noqa: F811
    """Lists of eight utterances and of a few more, which take over a row: stretches of labels on every frame (two-layer fp32 models: steps of one
    tile), stretches with a label every few frames up to one more than a last row's step holds, utterances that end one after the
    other, and (fp32) a large one, whose neighbours' operands are computed once more."""
    w = model_inputs(H, J, V1, L, B=8 * teams + more, T=67, seed=H + more, F=(J + 15) // 16 * 16, **extra)
    want = 60.0 * np.maximum(w.model.w_out[w.model.dims.blank].astype(np.float64), 0.0) - w.model.b_enc
    blank = np.linalg.lstsq(w.model.w_enc.astype(np.float64), want, rcond=None)[0].astype(np.float32)
    g = np.random.default_rng(w.B)
    gap = np.array([1, 2, 4, 5, 6, 8, 31, 32])[g.integers(0, 8, (w.B, 67))].cumsum(1)
    label = (gap[:, :, None] == np.arange(67)[None, None, :] + 1).any(1)
    label[g.random(w.B) < 0.4, :25] = True
    x = np.where(label[:, :, None], w.enc_out, blank[None, None]).astype(np.float32)
    if not bf16:
        x[3] *= np.float32(1e9)
    length = np.sort(g.integers(1, 68, w.B))[::-1].astype(np.int32)
    w = dataclasses.replace(w, enc_out=x, enc_len=length)
    eng = pkg.Engine(w.model, w.B, w.T, flags=pkg.RNNT_FLAG_BF16_ARITHMETIC if bf16 else 0)
    _, _, stats = check(pkg, w, w.variant, f"eight rows {H}/{J}/{V1}/{L} {extra} bf16={bf16} {more}", engine=eng, bf16=bf16, logp=not bf16)
    assert stats["n_teams"] == teams and stats["lookahead"] == 4
    eng.close()


# frames of a list (padded ones, as the host counts) from which on eight rows are worth it
@pytest.mark.parametrize("H,J,V1,L,bf16,teams,frames", [(64, 68, 60, 1, False, 32, 200), (324, 332, 1040, 1, True, 8, 200), (100, 128, 250, 2, False, 24, 240),
                                                        (128, 128, 257, 2, True, 32, 240), (320, 320, 500, 2, False, 12, 400), (324, 332, 1040, 2, True, 8, 400)])
def test_short_lists_stay_with_four_rows(pkg, H, J, V1, L, bf16, teams, frames):  # noqa: F811
    for T in (frames // 8 - 1, frames // 8):
        w = model_inputs(H, J, V1, L, B=8 * teams, T=T, seed=H + T)
        eng = pkg.Engine(w.model, w.B, w.T, flags=pkg.RNNT_FLAG_BF16_ARITHMETIC if bf16 else 0)
        _, _, stats = check(pkg, w, "label", f"short lists {H}/{J}/{V1}/{L} bf16={bf16} {T}", engine=eng, bf16=bf16, logp=not bf16)
        assert stats["n_teams"] == teams and stats["lookahead"] == (4 if 8 * T >= frames else 8)
        eng.close()


@pytest.mark.parametrize("H,J,V1,L,bf16,teams", EIGHT)
@pytest.mark.parametrize("extra", [{}, dict(durations=(0, 1, 3, 90)), dict(big_blanks=(2, 17, 70))])
@pytest.mark.parametrize("full", [False, True])
def test_one_utterance_a_team(pkg, H, J, V1, L, bf16, teams, extra, full):  # noqa: F811
    """One utterance, and as many as there are teams: labels that follow each other on a frame, at the first, last and one more than the last
    frame of a step, and none for several steps; empty utterances and such of a frame; jumps within a step and over several."""
    w = model_inputs(H, J, V1, L, B=teams if full else 1, T=131, seed=H + full, F=(J + 15) // 16 * 16, **extra)
    want = 60.0 * np.maximum(w.model.w_out[w.model.dims.blank].astype(np.float64), 0.0) - w.model.b_enc
    blank = np.linalg.lstsq(w.model.w_enc.astype(np.float64), want, rcond=None)[0].astype(np.float32)
    g = np.random.default_rng(w.B)
    gap = np.array([1, 2, 15, 16, 17, 33, 49])[g.integers(0, 7, (w.B, 131))].cumsum(1)
    label = (gap[:, :, None] == np.arange(131)[None, None, :] + 1).any(1)
    label[::3, 40:60] = True
    x = np.where(label[:, :, None], w.enc_out, blank[None, None]).astype(np.float32)
    length = np.sort(g.integers(60, 132, w.B))[::-1].astype(np.int32)
    if full:
        length[-1], length[-2] = 0, 1
        if not bf16:
            x[3] *= np.float32(1e9)
    w = dataclasses.replace(w, enc_out=x, enc_len=length)
    eng = pkg.Engine(w.model, w.B, w.T, flags=pkg.RNNT_FLAG_BF16_ARITHMETIC if bf16 else 0)
    _, _, stats = check(pkg, w, w.variant, f"one a team {H}/{J}/{V1}/{L} {extra} bf16={bf16} {full}", engine=eng, bf16=bf16, logp=not bf16)
    assert stats["n_teams"] == teams and stats["lookahead"] == 16
    eng.close()


def logits_in_64_bits(model, enc, tokens, frames, count):
    """Of every label that a decode emitted, after the labels before it."""
    import torch
    a = {k: torch.from_numpy(np.ascontiguousarray(v)).cuda().double() for k, v in model.arrays().items()}
    d, B = model.dims, enc.shape[0]
    h = [torch.zeros(B, d.H, dtype=torch.float64, device="cuda") for _ in range(d.L)]
    c, last, out = [v.clone() for v in h], torch.full((B,), d.blank, device="cuda"), []
    for i in range(int(count.max())):
        x = a["emb"][last]
        for l in range(d.L):
            g = (x @ a[f"w_ih{l}"].t() + a[f"b_ih{l}"] + h[l] @ a[f"w_hh{l}"].t() + a[f"b_hh{l}"]).chunk(4, 1)
            c[l] = torch.sigmoid(g[1]) * c[l] + torch.sigmoid(g[0]) * torch.tanh(g[2])
            x = h[l] = torch.sigmoid(g[3]) * torch.tanh(c[l])
        k, t = tokens[:, i].long().clamp(min=0), frames[:, i].long().clamp(min=0)
        z = torch.relu(enc[torch.arange(B, device="cuda"), t].double() @ a["w_enc"].t() + a["b_enc"] + x @ a["w_pred"].t() + a["b_pred"])
        out.append((z * a["w_out"][k]).sum(1) + a["b_out"][k])
        last = torch.where(i < count, k, last)
    return torch.stack(out, 1)


# rms over 48 models of what is left where high and low parts of a half block's weights have instructions of their own.  (The same on every run;
# 0.1 % above it is half of what the parts in one instruction cost layers of 320.)
@pytest.mark.parametrize("H,L,bias,rms", [(128, 1, 1.2, 1.10742e-7), (320, 1, 2.0, 2.25439e-7), (320, 2, 2.0, 2.04635e-7)])
def test_half_blocks_are_as_close_to_64_bits_as_whole_ones(pkg, H, L, bias, rms):  # noqa: F811
    """Models with the structure of a trained transducer: a label's embedding opposes its output row, and cell and projection pass that on."""
    import torch
    dims, n, square = synth.ModelDims(F=256, E=H, H=H, L=L, J=H, V1=257), 0, 0.0
    for seed in range(48):
        r = np.random.default_rng(seed)
        model = synth.make_model(dims, 0)
        for v in model.arrays().values():
            v[...] = (r.random(v.shape, dtype=np.float32) - np.float32(0.5)) * np.float32(0.2)
        model.emb[:-1] -= np.float32(5.0) * model.w_out[:-1]
        for l in range(L):
            model.w_ih[l][2 * H:3 * H] += np.float32(2.0) * np.eye(H, dtype=np.float32)
        model.w_pred[...] += np.float32(5.0) * np.eye(H, dtype=np.float32)
        model.b_out[-1] += np.float32(bias)
        g = torch.Generator(device="cuda").manual_seed(seed)
        enc = torch.randn((128, 200, dims.F), generator=g, device="cuda")
        eng = pkg.Engine(model, 128, 200)
        out = eng.decode("label", enc, torch.full((128,), 200, dtype=torch.int32, device="cuda"), 10)
        want = logits_in_64_bits(model, enc, out["tokens"], out["frames"], out["tok_len"])
        there = torch.arange(want.shape[1], device="cuda") < out["tok_len"][:, None]
        off = (out["logits"][:, :want.shape[1]].double() - want)[there]
        n, square = n + off.numel(), square + float((off * off).sum())
        eng.close()
    print(f"{H}/{L}: {n} labels, rms {np.sqrt(square / n):.5e}", flush=True)
    assert n > 200000 and np.sqrt(square / n) <= 1.001 * rms


# (the folded embedding table: tiles of 64 labels and 16 units, 32 values of the embedding at a time)
@pytest.mark.parametrize("H,J,V1,E", [(64, 60, 65, 1), (68, 64, 64, 31), (60, 128, 63, 32), (316, 320, 129, 33), (644, 640, 40, 65), (20, 72, 191, 96)])
@pytest.mark.parametrize("bf16", [False, True])
def test_folded_embedding_table(pkg, H, J, V1, E, bf16):  # noqa: F811
    dims = synth.ModelDims(F=32, E=E, H=H, L=1, J=J, V1=V1)
    model = synth.make_model(dims, H + V1, weight_range=0.15, emb_gain=4.0, pred_gain=3.0, blank_bias=1.5)
    x, ln = synth.make_inputs(E, 40, 30, dims.F, 0, 30)
    w = synth.Workload(f"folded table {H}/{V1}/{E}", "label", model, x, ln, 4)
    eng = pkg.Engine(model, w.B, w.T, flags=pkg.RNNT_FLAG_BF16_ARITHMETIC if bf16 else 0)
    check(pkg, w, "label", w.name, engine=eng, bf16=bf16, logp=True)
    eng.close()
