"""The decode kernel of one work-group per utterance: the narrowest and widest models it takes, one and two pairs of column
tiles, more utterances than work-groups, frames that go round its ring of 128, skips over whole chunks of them, and every
output, against the oracle."""
import dataclasses

import numpy as np
import pytest

import oracle
import synth
from parity_util import compare, to_lists
from test_gpu_parity import N_THREADS, check, pkg  # noqa: F401  (pkg: fixture)
from test_gpu_resident import model_inputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# (H, J, V1): outputs that just fill one to four tiles of 16 and one more or less, with the durations or big blanks
SHAPES = [(4, 4, 2), (64, 64, 17), (60, 64, 28), (64, 60, 29), (8, 52, 32), (64, 64, 33), (36, 64, 60), (64, 64, 64),
          (64, 64, 12), (60, 64, 15), (64, 52, 16), (64, 64, 44), (32, 64, 48), (64, 64, 49)]


@pytest.mark.parametrize("H,J,V1", SHAPES)
@pytest.mark.parametrize("extra", [{}, dict(durations=(0, 1, 3, 90)), dict(big_blanks=(2, 70, 300, 5))])
def test_shapes_and_decoders(pkg, H, J, V1, extra):  # noqa: F811
    if extra and V1 > 60:
        V1 = 60
    for B, T in ((1, 3), (7, 131), (300, 12)):
        w = model_inputs(H, J, V1, 1, B=B, T=T, seed=H + J + V1 + B, **extra)
        eng = pkg.Engine(w.model, w.B, w.T)
        _, _, stats = check(pkg, w, w.variant, f"solo {H}/{J}/{V1} {extra} {B}", engine=eng, logp=True)
        assert stats["team_size"] == 1
        if not extra:
            check(pkg, w, "frame", f"solo {H}/{J}/{V1} {B}", engine=eng)
        eng.close()


@pytest.mark.parametrize("V1,extra", [(17, {}), (33, {}), (49, {}), (45, dict(big_blanks=(2, 70, 300, 5))), (13, dict(big_blanks=(2, 70, 300, 5))), (29, dict(big_blanks=(2, 70, 300, 5)))])
def test_an_output_behind_the_tiles(pkg, V1, extra):  # noqa: F811
    """The 17th, 33rd or 49th output, a blank, beside outputs of the tiles: as large as one of them it loses, as the higher number; one bit
    above it wins.  (Rows of zeros: these outputs are their biases, exactly.)"""
    w = model_inputs(64, 64, V1, 1, B=5, T=40, seed=V1, **extra)
    check(pkg, w, w.variant, f"behind the tiles {V1} {extra}", logp=True)
    last = w.model.w_out.shape[0] - 1
    assert last in (16, 32, 48)
    for row in (0, 7, last - 5):
        w.model.w_out[[row, last]] = 0.0
        w.model.b_out[[row, last]] = np.float32(500.0)
        for above in (False, True):
            w.model.b_out[last] = np.nextafter(np.float32(500.0), np.float32(np.inf)) if above else np.float32(500.0)
            eng = pkg.Engine(w.model, w.B, w.T)
            out = eng.decode(w.variant, torch.from_numpy(w.enc_out).cuda(), torch.from_numpy(w.enc_len.astype(np.int32)).cuda(), 2)
            assert eng.stats()["team_size"] == 1
            n = out["tok_len"].cpu().numpy()
            assert np.array_equal(n, 0 * w.enc_len if above else 2 * w.enc_len)
            assert all((out["tokens"][b, :k] == row).all() for b, k in enumerate(n))
            eng.close()
        w.model.b_out[row] = -500.0


@pytest.mark.parametrize("T", [63, 64, 65, 127, 128, 129, 400])
@pytest.mark.parametrize("extra", [{}, dict(durations=(0, 1, 49, 64, 128)), dict(big_blanks=(15, 16, 17, 65))])
def test_frames_in_the_ring(pkg, T, extra):  # noqa: F811
    """Mostly blank frames, so that steps move on by sixteen; every length around a chunk's end."""
    w = model_inputs(64, 64, 20, 1, B=9, T=T, seed=T, F=64, **extra)
    want = 60.0 * np.maximum(w.model.w_out[w.model.dims.blank].astype(np.float64), 0.0) - w.model.b_enc
    blank = np.linalg.lstsq(w.model.w_enc.astype(np.float64), want, rcond=None)[0].astype(np.float32)
    g = np.random.default_rng(T)
    x = np.where(g.random((9, T, 1)) < 0.1, w.enc_out, blank[None, None]).astype(np.float32)
    w = dataclasses.replace(w, enc_out=x, enc_len=np.array([T, T - 1, T - 2, 0, 1, 16, 17, T // 2, min(T, 65)], dtype=np.int32))
    eng = pkg.Engine(w.model, w.B, w.T)
    check(pkg, w, w.variant, f"ring {T} {extra}", engine=eng, logp=True)
    eng.close()


def test_what_a_call_leaves(pkg):  # noqa: F811
    """Rows that are too short for their labels, lengths out of range, flags, the entry point without allocations, a smaller
    call after a larger one, a replayed graph, and weights that are not finite."""
    w = model_inputs(64, 64, 17, 1, B=40, T=30, seed=5)
    eng = pkg.Engine(w.model, w.B, w.T)
    ref, got, _ = check(pkg, w, "label", "solo", engine=eng)
    enc, ln = torch.from_numpy(w.enc_out).cuda(), torch.from_numpy(w.enc_len.astype(np.int32)).cuda()
    want = eng.decode("label", enc, ln, 4)
    want = {k: v.cpu().numpy() for k, v in want.items()}
    other = eng.decode("label_noalloc", enc, ln, 4)
    assert all(np.array_equal(other[k].cpu().numpy(), want[k]) for k in want)
    small = eng.decode("label", enc[:3].contiguous(), ln[:3].contiguous(), 4)
    n = small["tokens"].shape[1]
    assert np.array_equal(small["tokens"].cpu().numpy(), want["tokens"][:3, :n]) and eng.stats()["joint_samples"] > 0
    # out of range lengths, and room for two labels a row
    bad = ln.clone()
    bad[0], bad[1] = -3, 31
    tokens = torch.full((40, 2), 7, dtype=torch.int32, device="cuda")
    count = torch.zeros(40, dtype=torch.int32, device="cuda")
    done = torch.zeros(40, dtype=torch.int32, device="cuda")
    pkg.rnnt_engine_set_done_flags(eng.handle, done)
    pkg.rnnt_label_looping_decode(eng.handle, enc, bad, 40, 30, 4, tokens, count, 2,
                                  stream=torch.cuda.current_stream().cuda_stream)
    assert eng.status() == 3 and int(done.sum()) == 40
    full = eng.decode("label", enc, bad.clamp(0, 30), 4)
    assert torch.equal(count, full["tok_len"]) and torch.equal(tokens, full["tokens"][:, :2])
    pkg.rnnt_engine_set_done_flags(eng.handle, None)
    # a captured call
    out = {k: torch.from_numpy(v).cuda() for k, v in want.items()}
    stream = torch.cuda.Stream()
    cap = out["tokens"].shape[1]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        pkg.rnnt_label_looping_decode(eng.handle, enc, ln, 40, 30, 4, out["tokens"], out["tok_len"], cap, out["frames"],
                                      out["logits"], stream=torch.cuda.current_stream().cuda_stream)
    for i in range(3):
        for v in out.values():
            v.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert all(np.array_equal(out[k].cpu().numpy(), want[k]) for k in ("tokens", "tok_len", "frames", "logits")), i
    eng.close()
    w.model.w_out[3, 5] = np.inf
    eng = pkg.Engine(w.model, w.B, w.T)
    eng.decode("label", enc, ln, 4)
    assert eng.stats()["team_size"] != 1
    eng.close()


@pytest.mark.parametrize("durations,skipped", [((), 1), ((1, 2), 1), ((3, 2, 1), 3)])
def test_a_frame_whose_outputs_are_no_numbers_is_a_blank(pkg, durations, skipped):  # noqa: F811
    """An infinite value of a frame makes every output of it NaN: it has no label, and the frames around it are as without it.  (TDT:
    it moves on by the first duration.)"""
    w = model_inputs(64, 64, 17, 1, B=5, T=20, seed=3, durations=durations)
    w.model.b_out[w.model.dims.blank] -= 1.3          # (labels on a part of the frames)
    x, ln = w.enc_out.copy(), np.maximum(w.enc_len, 5)
    x[:, 3, 0] = np.inf
    at = 0 if durations else 3           # (TDT: the first frame, as no label goes past it)
    x, ln = np.ascontiguousarray(x[:, 3 - at:]), ln - (3 - at)
    eng = pkg.Engine(w.model, w.B, w.T)

    def run(a, n):
        out = eng.decode(w.variant, torch.from_numpy(a).cuda(), torch.from_numpy(n.astype(np.int32)).cuda(), 4)
        return {k: v.cpu().numpy() for k, v in out.items()}

    got, want = run(x, ln), run(np.ascontiguousarray(np.delete(x, range(at, at + skipped), axis=1)), np.maximum(ln - skipped, 0))
    assert np.array_equal(got["tok_len"], want["tok_len"]) and got["tok_len"].max() > 0
    for b, n in enumerate(got["tok_len"]):
        assert np.array_equal(got["tokens"][b, :n], want["tokens"][b, :n])
        f = want["frames"][b, :n]
        assert np.array_equal(got["frames"][b, :n], f + skipped * (f >= at))
    eng.close()


@pytest.mark.parametrize("cooperative", [False, True])
def test_decodes_of_other_engines_come_after(pkg, cooperative):  # noqa: F811
    """Decodes of a device run one after another, whatever their engines and streams: what is copied behind a short call on one
    stream is the finished result of a long call on another, where either, or both, are this kernel's."""
    flags = pkg.RNNT_FLAG_COOPERATIVE_LAUNCH if cooperative else 0
    small, wide = (64, 64, 17, 1), (324, 332, 520, 2)
    streams = torch.cuda.Stream(), torch.cuda.Stream()
    for first, then in ((small, small), (small, wide), (wide, small)):
        ws = [model_inputs(*first, B=4, T=4000, seed=8), model_inputs(*then, B=2, T=6, seed=9)]
        ws = [dataclasses.replace(w, enc_len=np.full(w.B, w.T, dtype=np.int32)) for w in ws]
        for w in ws:
            w.model.b_out[w.model.dims.blank] -= 4.0          # (labels on most frames: the long call takes milliseconds)
        engines = [pkg.Engine(w.model, w.B, w.T, flags=flags) for w in ws]
        calls = []
        for w, eng in zip(ws, engines):
            out = eng.alloc_outputs(w.B, w.T * w.max_symbols)
            out["tok_len"].fill_(-1)
            calls.append((eng, torch.from_numpy(w.enc_out).cuda(), torch.from_numpy(w.enc_len).cuda(), out))
        there = torch.full_like(calls[0][3]["tok_len"], -2)
        torch.cuda.synchronize()
        for stream, w, (eng, enc, ln, out) in zip(streams, ws, calls):
            with torch.cuda.stream(stream):
                eng.decode("label", enc, ln, w.max_symbols, out=out)
        with torch.cuda.stream(streams[1]):
            there.copy_(calls[0][3]["tok_len"])
        torch.cuda.synchronize()
        for w, (eng, _, _, out) in zip(ws, calls):
            assert eng.status() == 0
            net = oracle.LstmNet(w.model)
            ref = oracle.decode(net, w.enc_out, w.enc_len, w.max_symbols, "seq", n_threads=N_THREADS)
            compare(w, net, ref, to_lists(out, w.B), w.max_symbols)
            eng.close()
        assert torch.equal(there, calls[0][3]["tok_len"]) and int(there.min()) > 1000, (first, then, there)
