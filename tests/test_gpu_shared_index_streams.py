"""Steps that are alive together on one training stream share their index streams: each has to leave
what it leaves alone, bit for bit, whatever the others do, also from two threads and when another is
closed early; closing one does not wait for another, and steps on different training streams do not
wait for each other's data."""
import threading

import pytest
import torch

pytestmark = pytest.mark.gpu

# (tables, rows, dim, batch, bag): one index stream; three of them with issue threads; two
SHAPES = [(3, 5000, 16, 300, 2), (1, 20000, 8, 20000, 1), (12, 3000, 4, 25000, 1)]
N, K = 23, 5


def _make(shape, seed):
    from paper_2404_04270_amd.step import PipelinedStep
    T, R, D, B, L = shape
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    weights = [torch.rand(R, D, device="cuda", generator=gen) for _ in range(T)]
    hot = [torch.arange(0, R, 7, dtype=torch.int32, device="cuda") for _ in range(T)]
    idx = [(torch.rand(T, B, L, device="cuda", generator=gen) ** 4 * R).int() for _ in range(N)]
    grad = torch.randn(T, B, D, device="cuda", generator=gen)
    torch.cuda.synchronize()
    return PipelinedStep(weights, hot, B, L, 0.01, 0.05, K), idx, grad


def _batches(step, idx, grad, count=N):
    ahead = 0
    for k in range(count):
        while ahead < count and step.room() > 0:
            step.submit(idx[ahead])
            ahead += 1
        step.forward()
        step.backward(grad)
        yield


def _result(step):
    step.flush()
    torch.cuda.synchronize()
    return [w.clone() for w in step.tables.weights] + [b.clone() for b in step.bits]


def _alone(k):
    step, idx, grad = _make(SHAPES[k], k)
    for _ in _batches(step, idx, grad):
        pass
    out = _result(step)
    step.close()
    return out


def _same(a, b):
    return all(torch.equal(x, y) for x, y in zip(a, b))


def test_steps_in_turn_and_one_closed_early():
    want = [_alone(k) for k in range(3)]
    made = [_make(s, k) for k, s in enumerate(SHAPES)]
    extra, idx, grad = _make(SHAPES[1], 9)
    runs = [_batches(*m) for m in made]
    other = _batches(extra, idx, grad)
    for k in range(N):
        for r in runs:
            next(r)
        if k < 4:
            next(other)
        if k == 4:
            extra.close()              # with batches submitted and not trained on
    assert all(_same(_result(m[0]), w) for m, w in zip(made, want))
    for m in made:
        m[0].close()
    assert _same(_alone(1), want[1])   # the streams are made again after the last was given back


@pytest.mark.parametrize("one_stream", [False, True])
def test_two_threads(one_stream):
    want = [_alone(k) for k in range(2)]
    got, errors = [None, None], []

    def work(k):
        try:
            with torch.cuda.stream(None if one_stream else torch.cuda.Stream()):
                step, idx, grad = _make(SHAPES[k], k)
                for _ in _batches(step, idx, grad):
                    pass
                got[k] = _result(step)
                step.close()
        except Exception as e:         # noqa: BLE001
            errors.append(e)

    threads = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    assert all(_same(g, w) for g, w in zip(got, want))


def _sleep_cycles(seconds):
    begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda._sleep(1000)
    begin.record()
    torch.cuda._sleep(1_000_000)
    end.record()
    end.synchronize()
    return int(1_000_000 * seconds * 1e3 / max(begin.elapsed_time(end), 1e-3))


def _late_event(cycles):
    """An event that happens once a stream of its own has slept."""
    event = torch.cuda.Event()
    with torch.cuda.stream(torch.cuda.Stream()):
        torch.cuda._sleep(cycles)
        event.record()
    return event


def test_closing_a_step_does_not_wait_for_the_data_of_another():
    cycles = _sleep_cycles(0.4)
    a, idx_a, grad_a = _make(SHAPES[0], 1)
    b, idx_b, grad_b = _make(SHAPES[0], 2)
    for _ in _batches(a, idx_a, grad_a, 3):
        pass
    torch.cuda.synchronize()
    late = _late_event(cycles)
    b.submit(idx_b[0], ready=late)
    b.flush()                          # the wait for `late` is on the streams both have
    a.close()
    assert not late.query()
    b.forward()
    b.backward(grad_b)
    torch.cuda.synchronize()
    b.close()


def test_steps_on_two_training_streams_do_not_wait_for_each_others_data():
    # Streams may share one of the GPU's few hardware queues and wait for each other there, so one
    # attempt of several, with streams on other queues each time, has to show it.
    cycles = _sleep_cycles(0.2)
    passed = []
    for k in range(8):
        main_a, main_b = torch.cuda.Stream(), torch.cuda.Stream()
        with torch.cuda.stream(main_a):
            a, idx_a, grad_a = _make(SHAPES[0], 1)
        with torch.cuda.stream(main_b):
            b, idx_b, grad_b = _make(SHAPES[0], 2)
        torch.cuda.synchronize()
        late = _late_event(cycles)
        a.submit(idx_a[0], ready=late)
        a.flush()
        with torch.cuda.stream(main_b):
            for _ in _batches(b, idx_b, grad_b, 3):
                pass
            trained = torch.cuda.Event()
            trained.record()
        trained.synchronize()
        passed.append(not late.query())
        with torch.cuda.stream(main_a):
            a.forward()
            a.backward(grad_a)
        torch.cuda.synchronize()
        a.close()
        b.close()
        if passed[-1]:
            break
    assert passed[-1], passed
