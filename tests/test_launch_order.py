"""What calls enqueue, read from the library's host side run against stand-ins of the HIP runtime (launch_trace.py,
hip_trace.c): no GPU needed, nothing is executed."""
import json
import os
import subprocess
import sys

import pytest

from helpers import PAIR_CASES, ROUNDS_CASE, pair_stream, rounds_stream
from paper_2211_10280_amd import binding as B

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def trace(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("hip_trace") / "hip_trace.so")
    subprocess.check_call(["gcc", "-O1", "-Wall", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "hip_trace.c")])
    lib = os.environ.get("TENSAIR_TRACED_LIB", B.LIB_PATH)

    def run(calls, tokens=1_000_000, counts=None, **model):
        model = {"row_stride": model["dim"], "dtype": B.F32, "max_peers": 0, "worker_id": 0, "seed": 7, "flags": 0, **model}
        r = subprocess.run([sys.executable, os.path.join(HERE, "launch_trace.py"), lib, so], capture_output=True, text=True,
                           input=json.dumps({"model": model, "tokens": tokens, "counts": counts, "calls": calls}), timeout=120)
        assert r.returncode == 0, r.stderr
        return json.loads(r.stdout)

    return run


def launches(did):
    """[(kernel, workgroups, stream)] of one call, kernels without namespace and types"""
    out = []
    for d in did:
        if d[0] == "launch":
            n = int("".join(c for c in d[1][2:5] if c.isdigit()))            # _Z<length><name>...
            out.append((d[1][2 + len(str(n)):][:n], int(d[2]), d[4]))
    return out


def names(did):
    return [k for k, _, _ in launches(did)]


# 60 centers: chained preparation (8 tiles); 1500 centers: counted (188 tiles), forward pass on the second stream
SMALL = dict(vocab=50_000, dim=64, window=8, negatives=15, max_centers=6000)


@pytest.mark.parametrize("n", [60, 1500])
@pytest.mark.parametrize("kind", ["grad", "step"])
def test_calls_after_a_capture_rely_on_nothing_that_was_left(trace, kind, n):
    """A recorded call has not run when the next one is enqueued, and runs again later: neither may count on counters,
    masks or a mini-batch that the other is to leave in the workspace."""
    batch = lambda i: [i * n, n, 0]                                            # noqa: E731
    call = lambda i: [kind] + batch(i) + ([0] if kind == "step" else [])       # noqa: E731
    calls = [["prefetch"] + batch(0), ["prefetch"] + batch(1), call(0), ["capture", 1], call(1), ["capture", 0]]
    calls += [c for i in range(2, 8) for c in (["prefetch"] + batch(i), ["prefetch"] + batch(i + 1), call(i))]
    got = trace(calls, **SMALL)
    assert all(c["rc"] == 0 for c in got)
    assert [c["call"][0] for c in got[:4]] == ["prefetch", "prefetch", kind, kind]
    for c in got[3:]:
        did = names(c["did"])
        if c["call"][0] == "prefetch":
            assert did == []
        else:
            assert did.index("k_prep_clear") < did.index("k_prep_keys")        # digit counts zeroed by the call itself
            assert ("k_apply_clear" in did) == (kind == "step")                # and the masks of the update's index


def test_a_captured_step_without_pairs_carries_no_phase(trace):
    """The mini-batch whose phases ride is half prepared when a step of an empty one is recorded: none of them may ride
    with its update, which does not run now."""
    batch = lambda i: [i * 60, 60, 0]                                          # noqa: E731
    calls = [["prefetch"] + batch(0), ["prefetch"] + batch(1), ["step"] + batch(0) + [0], ["capture", 1], ["step", 60, 0, 0, 0],
             ["capture", 0], ["step"] + batch(1) + [0]]
    got = trace(calls, **dict(SMALL, vocab=300_000))                           # three passes: the segments have not ridden yet
    update = [launches(c["did"])[-1] for c in got[2:]]
    assert update[0][1] > update[1][1] and update[1] == update[2]              # the first carried a pass
    assert "k_prep_keys" in names(got[4]["did"])


def test_an_update_that_is_captured_leaves_no_mask_clean(trace):
    got = trace([["step", 0, 60, 0, 0], ["step", 60, 60, 0, 0], ["capture", 1], ["apply", 60, 900, 0], ["capture", 0],
                 ["step", 120, 60, 0, 0], ["step", 180, 60, 0, 0]], **SMALL)
    assert "k_apply_clear" not in names(got[1]["did"])                         # cleared during the step before
    assert all("k_apply_clear" in names(c["did"]) for c in got[3:])


@pytest.mark.parametrize("V", [B.MAX_VOCAB, B.MAX_VOCAB - 16 * 600])
def test_no_launch_grows_beyond_its_limit_in_the_largest_vocabulary(trace, V):
    """2^32 threads: the update of the largest vocabulary fills a launch, so a phase rides with it only where there is
    room (each of the two sizes is on its side of that)."""
    step = lambda i: ["step", 1000 * i, 1000, 0, 0]                            # noqa: E731
    calls = [step(0), ["prefetch", 1000, 1000, 0], ["prefetch", 2000, 1000, 0], step(1), ["prefetch", 3000, 1000, 0], step(2)]
    got = trace(calls, vocab=V, dim=256, window=8, negatives=15, max_centers=800_000, dtype=B.BF16)
    grids = [g for c in got if c["call"][0] == "step" for k, g, _ in launches(c["did"]) if k == "k_apply"]
    assert len(grids) == 3 and grids[0] == (V + 63) // 64 * 4
    assert all(d[0] != "launch" or int(d[2]) * int(d[3]) < 1 << 32 for c in got for d in c["did"])
    assert (grids[2] > grids[0]) == (V < B.MAX_VOCAB)                          # a phase rode along


@pytest.mark.parametrize("kind", ["grad", "step"])
def test_riding_goes_on_after_a_mini_batch_too_large_to_ride(trace, kind):
    """628 tiles, then 201 each, announced two deep: the first is prepared by its own call; from there on the next one
    rides in the launches of the call before, and a call has nothing, or little, of its own left to prepare."""
    sizes = [5000, 5000] + [1600] * 5
    calls = []
    for i, n in enumerate(sizes):
        calls += [["prefetch", 5000 * (i + 1), m, 0] for m in sizes[i + 1:i + 2]]
        calls.append([kind, 5000 * i, n, 0] + ([0] if kind == "step" else []))
    calls.insert(0, ["prefetch", 0, 5000, 0])
    got = [c for c in trace(calls, **SMALL) if c["call"][0] == kind]
    prep = [[k for k in names(c["did"]) if k.startswith("k_prep")] for c in got]
    assert prep[0].count("k_prep_count") == 2 and prep[1].count("k_prep_count") == 2
    assert prep[1].count("k_prep_keys") == 2                                   # its own, and the next one's
    for p in prep[2:]:
        assert p == [] or (kind == "grad" and p == ["k_prep_segments"]), p


@pytest.mark.parametrize("kind", ["grad", "step"])
def test_mini_batches_of_medium_size_are_prepared_beside_the_call_before(trace, kind):
    """302 tiles, announced two deep, no long update to follow: on the library's stream, which starts with the forward
    pass of the call before; the call that consumes one waits for its keys, and before the reduction for the rest."""
    batch = lambda i: [2400 * i, 2400, 0]                                      # noqa: E731
    calls = [["prefetch"] + batch(0)]
    for i in range(5):
        calls += [["prefetch"] + batch(i + 1), [kind] + batch(i) + ([0] if kind == "step" else [])]
    got = [c["did"] for c in trace(calls, **SMALL) if c["call"][0] == kind]
    for i, did in enumerate(got[:-1]):
        side = [k for k, _, s in launches(did) if s != "0"]
        assert side == ["k_prep_clear"] * (i < 1) + ["k_prep_keys"] + ["k_prep_count", "k_prep_pass"] * 2 + ["k_prep_segments"] * 2
        assert not any(k.startswith("k_prep") for k, _, s in launches(did) if s == "0")
        at = {k: j for j, d in enumerate(did) if d[0] == "launch" and d[4] == "0" for k in ("forward", "segreduce") if k in d[1]}
        keys = next(j for j, d in enumerate(did) if d[0] == "launch" and "k_prep_keys" in d[1])
        fork = next(j for j, d in enumerate(did) if d[0] == "wait" and d[1] != "0")
        assert fork < at["forward"] and fork < keys
        mine = [j for j, d in enumerate(did) if d[0] == "wait" and d[1] == "0"]
        assert mine[0] < at["forward"] < mine[1] < keys and mine[1] < at["segreduce"]


@pytest.mark.parametrize("kind", ["grad", "step"])
def test_what_is_announced_one_at_a_time_is_prepared_at_once(trace, kind):
    """60 centers (8 tiles): on the caller's stream, all but the last phase, without an event.  1500 (188 tiles): on the
    library's stream; the forward pass that consumes it waits for its keys, the reduction for the rest."""
    calls = []
    for i, n in enumerate([60, 1500] * 2):
        calls += [["prefetch", 2000 * i, n, 0], [kind, 2000 * i, n, 0] + ([0] if kind == "step" else [])]
    got = trace(calls, **SMALL)
    for ahead, call in zip(got[::2], got[1::2]):
        did, events = launches(ahead["did"]), [d for d in ahead["did"] if d[0] != "launch"]
        prep = [k for k, _, _ in did if k != "k_prep_clear"]
        assert not any(k.startswith("k_prep") for k in names(call["did"]))     # the segments ride
        forward = next(i for i, d in enumerate(call["did"]) if d[0] == "launch" and "k_forward" in d[1])
        reduction = next(i for i, d in enumerate(call["did"]) if d[0] == "launch" and "k_segreduce" in d[1])
        waits = [(i, d[2]) for i, d in enumerate(call["did"]) if d[0] == "wait"]
        if ahead["call"][2] == 60:
            assert prep == ["k_prep_keys", "k_prep_pass", "k_prep_pass"] and {s for _, _, s in did} == {"0"}
            assert not events and not waits
        else:
            assert prep == ["k_prep_keys"] + ["k_prep_count", "k_prep_pass"] * 2 + ["k_prep_segments"] * 2
            assert len({s for _, _, s in did}) == 1 and "0" not in {s for _, _, s in did}
            order = ["event" if d[0] == "event" else d[1] for d in ahead["did"] if d[0] != "wait"]
            recorded = [d[1] for d in events if d[0] == "event"]               # fork, keys, all
            assert len(recorded) == 3 and "k_prep_keys" in order[order.index("event", 1) - 1]
            assert [w for _, w in waits] == recorded[1:]
            assert waits[0][0] < forward < waits[1][0] < reduction


def test_long_key_lists_are_not_counted_by_every_tile(trace):
    """From 41 groups of tiles on, the groups' counts are summed once per pass, in a launch of their own: work per
    occurrence does not grow with the mini-batch."""
    model = dict(SMALL, max_centers=80_000)
    got = trace([["grad", 100, n, 0] for n in (20_480, 20_481, 80_000)], **model)
    prep = [[k for k in names(c["did"]) if k in ("k_prep_count", "k_prep_scan", "k_prep_pass")] for c in got]
    assert prep[0] == ["k_prep_count", "k_prep_pass"] * 2
    assert prep[1] == prep[2] == ["k_prep_count", "k_prep_scan", "k_prep_pass"] * 2


@pytest.mark.parametrize("V,D,dtype,rows", [                  # vocabulary rows per workgroup of four waves
    (262_143, 132, B.F32, 16), (262_144, 132, B.F32, 64), (393_215, 300, B.F32, 16), (393_216, 300, B.F32, 64),
    (655_359, 1024, B.F32, 16), (655_360, 1024, B.F32, 64), (147_455, 132, B.BF16, 16), (147_456, 132, B.BF16, 64),
    (221_183, 300, B.BF16, 16), (221_184, 300, B.BF16, 64), (655_359, 100, B.F32, 32), (655_360, 100, B.F32, 128),
    (655_360, 64, B.F32, 128), (4_000_000, 32, B.F32, 128)])
def test_rows_per_wave_where_few_are_touched(trace, V, D, dtype, rows):
    """A quarter of a row of capacity per vocabulary row: the sparse shape of the update from the vocabulary on that its
    own and the dense shape were measured to take the same time at."""
    model = dict(SMALL, vocab=V, dim=D, dtype=dtype, max_centers=64, max_peers=1)
    got = launches(trace([["apply", 60, V // 8, 1]], **model)[0]["did"])[-1]
    assert got[0] == ("k_apply" if D > 128 else "k_apply_sub")
    assert got[1] == ((V + 63) // 64 * 64 + rows - 1) // rows


@pytest.mark.parametrize("outputs", [[], ["negatives"], ["offsets_in"], ["offsets_out"], ["negatives", "offsets_in", "offsets_out"]])
def test_optional_outputs_do_not_choose_the_gradients_form(trace, outputs):
    """A large mini-batch over a small vocabulary goes by pairs of words whatever else is asked for; its occurrences are
    sorted only for their offsets."""
    did = launches(trace([["grad", 100, 5000, 0] + outputs], vocab=300, dim=64, window=8, negatives=15, max_centers=5000)[0]["did"])
    assert "k_group_rows" in [k for k, _, _ in did] and not any("forward" in k or "segreduce" in k for k, _, _ in did)
    tiles = [g for k, g, _ in did if k == "k_prep_pass"]
    assert tiles == [3 + (625 if "offsets_out" in outputs else 0)]


def test_stages_of_the_gradient_by_pairs_are_timed_one_by_one(trace):
    """Profile level 2: an event before the first stage and after every one, each in launches of its own."""
    did = trace([["profile", 2], ["grad", 100, 5000, 0]], vocab=300, dim=64, window=8, negatives=15, max_centers=5000)[1]["did"]
    stages = [[]]
    for d in did:
        if d[0] == "event":
            stages.append([])
        else:
            stages[-1] += names([d])
    assert stages == [[], ["k_prep_clear", "k_prep_keys"], ["k_prep_count", "k_prep_pass"], ["k_prep_segments"] * 2,
                      ["k_group_count", "k_group_rows"], ["k_group_reduce"], ["k_group_any", "k_group_reduce"], []]


# by pairs of words: the most frequent word's share of the negatives is counts^0.75 / sum
@pytest.mark.parametrize("counts,pairs", [([7], False), ([1, 1], True), ([2, 1], False), ([100, 46, 30, 22], True), ([2000] + [1] * 200, False),
                                          ([20] + [1] * 299, True)])
def test_a_word_that_is_most_of_the_negatives_is_not_counted_by_pairs(trace, counts, pairs):
    did = names(trace([["grad", 100, 5000, 0]], counts=counts, vocab=len(counts), dim=64, window=8, negatives=15, max_centers=5000)[0]["did"])
    assert ("k_group_rows" in did) == pairs and any("forward" in k for k in did) != pairs


@pytest.mark.parametrize("V,D,n,others,rides", [
    (300, 132, 2500, 64, True), (300, 132, 2500, 1000, False),        # the update of small tables is as short as the chaining
    (300, 64, 2500, 64, False),                                       # narrow rows are chained faster
    (60_000, 132, 2500, 4, False), (60_000, 132, 5000, 4, True)])     # a larger update hides a phase, unless the chain is long
def test_a_phase_rides_with_the_chaining_of_long_rows_where_that_takes_longer(trace, V, D, n, others, rides):
    """One word a thousand times, the others `others` times each: 0.18 occurrences per pair (139 tiles of 32 in 25 000 pairs), 0.02
    (16) and, among a thousand words, 0.5 (387, and 774 in 50 000 pairs)."""
    counts = [1000] + [others] * (min(V, 1000) - 1)
    batch = lambda i: [n * i, n, 0]                                            # noqa: E731
    calls = [["prefetch"] + batch(0)]
    for i in range(4):
        calls += [["prefetch"] + batch(i + 1), ["step"] + batch(i) + [0]]
    model = dict(counts=counts, vocab=V, dim=D, window=5, negatives=5, max_centers=n)
    chaining = lambda c: [g for k, g, _ in launches(c["did"]) if k == "k_segfixup"]     # noqa: E731
    got = [g for c in trace(calls, **model) if c["call"][0] == "step" for g in chaining(c)]
    alone = chaining(trace([["grad", 0, n, 0]], **model)[0])[0]
    assert len(got) == 4 and [g > alone for g in got[:3]] == [rides] * 3


# words, rows, table, centers and negatives on both sides of a border: phases of the preparation (2^18 words), streamed tables (2^30
# bytes), elements of a row (512), occurrences (131 072), partials of the longest row expected (16 times 32, times rows side by side; 4
# times where the table has at most 2^19 elements of wide rows, 8 times up to 2^21)
@pytest.mark.parametrize("V,D,stride,dtype,n,N,most,chains", [
    (262_144, 64, 64, B.F32, 60, 5, 1, True), (262_145, 64, 64, B.F32, 60, 5, 1, False), (250_000, 512, 536, B.F32, 60, 5, 1, True),
    (250_000, 512, 540, B.F32, 60, 5, 1, False), (250_000, 512, 540, B.BF16, 60, 5, 1, True), (50_000, 512, 512, B.F32, 60, 5, 1, True),
    (50_000, 516, 516, B.F32, 60, 5, 1, False), (50_000, 64, 64, B.F32, 1638, 7, 1, True), (50_000, 64, 64, B.F32, 1640, 7, 1, False),
    (1_000, 300, 300, B.F32, 1600, 7, 50, True), (1_000, 300, 300, B.F32, 1600, 7, 150, False), (1_800, 300, 300, B.F32, 1600, 7, 150, True),
    (1_800, 300, 300, B.F32, 1600, 7, 250, False), (6_990, 300, 300, B.F32, 1600, 7, 250, False), (6_992, 300, 300, B.F32, 1600, 7, 250, True),
    (1_800, 300, 300, B.F32, 1600, 7, 1500, False), (1_000, 128, 128, B.F32, 1600, 7, 1500, True)])
def test_small_steps_chain_long_rows_in_their_update(trace, V, D, stride, dtype, n, N, most, chains):
    got = trace([["step", 100, n, 0, 1], ["grad", 9_000, n, 0]], counts=[10 * most] + [10] * (min(V, 1000) - 1), vocab=V, dim=D, row_stride=stride,
                dtype=dtype, window=5, negatives=N, max_centers=n, max_peers=1)
    assert ["k_segfixup" in names(c["did"]) for c in got] == [not chains, True]


# with messages, on both sides: words (131 072 with narrow rows, 196 608 with bfloat16 tables and rows of up to 256 elements, of which
# few are touched), elements of a row, rows of capacity (a fifth of the words; the own gradient has 3 600)
@pytest.mark.parametrize("V,D,dtype,rows,chains", [
    (131_072, 128, B.F32, 100, True), (131_073, 128, B.F32, 100, False), (131_073, 132, B.F32, 100, True), (262_144, 132, B.F32, 100, True),
    (196_608, 132, B.BF16, 100, True), (196_609, 132, B.BF16, 100, False), (196_609, 256, B.BF16, 100, False), (196_609, 260, B.BF16, 100, True),
    (200_000, 200, B.BF16, 36_399, False), (200_000, 200, B.BF16, 36_400, True)])
def test_small_steps_with_messages_chain_long_rows_in_their_update(trace, V, D, dtype, rows, chains):
    got = trace([["step_packed", 100, 60, 0, 1, rows]], vocab=V, dim=D, dtype=dtype, window=5, negatives=5, max_centers=60, max_peers=1)
    assert got[0]["rc"] == 0 and ("k_segfixup" in names(got[0]["did"])) == (not chains)


@pytest.mark.parametrize("case", PAIR_CASES, ids=lambda c: f"V{c[0]}_D{c[1]}_B{c[6]}_{c[8]}")
def test_the_cases_of_the_gradient_by_pairs_go_by_pairs(trace, case):
    V, D, stride, _, w, N, n, begin, dtype = case
    tok, counts = pair_stream(case)
    did = names(trace([["grad", begin, n, 0]], tokens=len(tok), counts=counts.tolist(), vocab=V, dim=D, row_stride=stride, window=w,
                      negatives=N, max_centers=n, dtype=B.F32 if dtype == "f32" else B.BF16)[0]["did"])
    assert [k for k in did if k.startswith("k_group")] == ["k_group_count", "k_group_rows", "k_group_any", "k_group_reduce"]


@pytest.mark.parametrize("D,dtype", [(64, B.F32), (260, B.BF16), (516, B.F32)])
def test_the_case_of_many_frequent_words_goes_by_pairs(trace, D, dtype):
    V, w, N, n, begin = ROUNDS_CASE
    tok, counts = rounds_stream()
    did = names(trace([["grad", begin, n, 0]], tokens=len(tok), counts=counts.tolist(), vocab=V, dim=D, window=w, negatives=N, max_centers=n,
                      dtype=dtype)[0]["did"])
    assert "k_group_rows" in did


# words, rows, window, negatives, centers on both sides of a border, the Zipf exponent of the counts: occurrences in all (2^20), tasks per
# position (128 and 512), words (12 288), occurrences per word by width of the rows, tasks and how much positions repeat words
@pytest.mark.parametrize("V,D,w,N,below,above,zipf", [
    (300, 64, 8, 15, 4096, 4097, 1.1), (300, 300, 1, 62, 20_000, None, 1.1), (300, 300, 1, 63, None, 20_000, 1.1),
    (300, 300, 8, 31, None, 2100, 1.1), (300, 300, 8, 32, 2100, None, 1.1), (12_288, 300, 8, 15, None, 4097, 1.5), (12_289, 300, 8, 15, 9000, None, 1.5),
    (12_000, 64, 8, 15, 9374, 9375, 1.5), (12_000, 68, 8, 15, 7031, 7032, 1.5), (12_000, 132, 8, 15, 6374, 6375, 1.5),
    (12_000, 64, 8, 15, 7031, 7032, 1.2), (12_000, 132, 8, 7, 9749, 9750, 1.2), (12_000, 132, 8, 15, 4218, 4219, 1.2),
    (12_000, 256, 8, 15, 4218, 4219, 1.2), (12_000, 260, 8, 15, 4096, 4097, 1.2)])
def test_borders_of_the_gradient_by_pairs(trace, V, D, w, N, below, above, zipf):
    counts = [max(1, round(2e6 * (i + 1) ** -zipf)) for i in range(V)]
    got = trace([["grad", 100, n, 0] for n in (below, above) if n], counts=counts, vocab=V, dim=D, window=w, negatives=N, max_centers=20_000)
    assert ["k_group_rows" in names(c["did"]) for c in got] == [False] * (below is not None) + [True] * (above is not None)


F, H = B.F32, B.BF16


@pytest.mark.parametrize("D,dtype,V,rows,sweeps", [            # rows: vocabulary rows per row of capacity, or the capacity itself
    (132, F, 131_071, 6, False), (132, F, 131_072, 6, True), (256, H, 524_287, 5.1, True), (256, F, 524_287, 4.9, False),
    (256, F, 524_288, 10.9, False), (256, H, 524_288, 11.1, True), (256, F, 999_999, 10.9, False), (256, F, 1_000_000, 5.1, True),
    (256, F, 4_000_000, 5.1, True), (260, H, 524_287, 5.1, True), (512, H, 524_288, 15.9, False), (512, H, 524_288, 16.1, True),
    (260, F, 655_359, 5.1, True), (512, F, 655_360, 15.9, False), (512, F, 999_999, 16.1, True), (512, F, 1_000_000, 31, False),
    (512, F, 1_000_000, 33, True), (512, H, 2_999_999, 31, False), (512, F, 3_000_000, 16.1, True), (300, F, 3_999_999, 15.9, False),
    (300, F, 4_000_000, 11.1, True), (300, F, 4_000_000, 10.9, False), (300, H, 4_000_000, 15.9, False), (516, F, 524_287, 6.9, False),
    (516, F, 524_287, 7.1, True), (1024, H, 999_999, 16.1, True), (1024, F, 1_000_000, 1000, False), (1024, F, 2_999_999, 1000, False),
    (1024, H, 3_000_000, 16.1, True), (128, F, 131_071, 6, False), (128, F, 131_072, 6, True), (128, H, 999_999, 5.1, True),
    (128, F, 1_000_000, 100, False), (64, F, 400_000, 28_000, True), (64, H, 400_000, 28_001, False), (36, F, 140_000, 5.1, True),
    (32, F, 299_999, 5.1, True), (32, F, 300_000, 5.1, False), (32, H, 300_000, 28_000, True)])
def test_borders_of_the_sweep_of_the_update(trace, D, dtype, V, rows, sweeps):
    """A sweep's grid is what fits the chip, 256 compute units times 7; the other shapes' covers the vocabulary."""
    rows = int(V / rows) if rows <= 1000 else rows
    did = trace([["apply", 60, rows, 0]], **dict(SMALL, vocab=V, dim=D, dtype=dtype, max_centers=64))[0]["did"]
    assert (launches(did)[-1][1] == 256 * 7) == sweeps
