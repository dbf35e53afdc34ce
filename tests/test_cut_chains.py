"""Flat clusters of dendrograms whose long chain avoids the merges that the stages of cluster_kernels.hip send up: the same labels, and the time of a
few passes over all merges, however deep the chain is."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    import paper_2306_16354_amd as slhc
    slhc.load_library()
    return slhc


def sent_up(group, bits):
    h = (group * 0x9e3779b1) & 0xffffffff
    h = ((h ^ (h >> 15)) * 0x85ebca6b) & 0xffffffff
    return (h ^ (h >> 13)) & ((1 << bits) - 1)


def in_stage(merges, stage):
    """Which merges are in `stage`: one of every eight is in the first, of those one of every sixteen in the next, and so on."""
    group, fine = np.arange(merges, dtype=np.int64), np.ones(merges, bool)
    for r in range(stage):
        bits = 3 if r == 0 else 4
        fine &= sent_up(group >> bits, bits) == (group & ((1 << bits) - 1))
        group >>= bits
    return fine


def chain(N, stage, pairs):
    """Merges of `stage` lie beside the chain that the others form; `pairs`: only merges that have no part in the chain have rows."""
    avoid, children, rows = in_stage(N - 1, stage), np.empty((N - 1, 2), np.int64), iter(range(N))
    last, beside = -1, []
    for i in range(N - 1):
        if pairs and i < N // 2:
            children[i] = next(rows), next(rows)
            beside.append(N + i)
            continue
        if pairs and (last < 0 or avoid[i]) and len(beside) > 2:
            a, b = beside.pop(), beside.pop()
            (beside.append(N + i) if avoid[i] else None)
            last = last if avoid[i] else N + i
        elif not pairs and avoid[i] and 2 * (N - 1 - i) > N // 16 + 2 * len(beside):
            a, b = next(rows), next(rows)
            beside.append(N + i)
        else:
            a = last if last >= 0 else next(rows)
            b = beside.pop() if beside else next(rows)
            last = N + i
        children[i] = min(a, b), max(a, b)
    return children


def cut(children, N, kept):
    top = list(range(N + kept))
    for i in range(kept - 1, -1, -1):
        a, b = children[i]
        top[a] = top[b] = top[N + i]
    return np.unique(np.array(top[:N]), return_inverse=True)[1]


def least_ms(f):
    least = float("inf")
    for _ in range(8):
        begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        begin.record()
        f()
        end.record()
        end.synchronize()
        least = min(least, begin.elapsed_time(end))
    return least


@pytest.mark.parametrize("N", [8200, 40_000, 300_000])
@pytest.mark.parametrize("stage", [1, 2, 3])
@pytest.mark.parametrize("pairs", [False, True])
def test_chain_beside_the_stages(lib, N, stage, pairs):
    children = chain(N, stage, pairs)
    flat = np.sort(children.ravel())
    assert np.array_equal(flat, np.r_[np.arange(2 * N - 2)]) and (children.max(1) < N + np.arange(N - 1)).all()       # every node but the last has one parent
    dev = torch.from_numpy(children.astype(np.int32)).cuda()
    plain = torch.from_numpy(np.stack([np.r_[0, N + np.arange(N - 2)], np.arange(1, N)], 1).astype(np.int32)).cuda()
    for kept in (N // 2 + 3, N - 500, N - 1):
        print(f"chain beside stage {stage} N={N} kept={kept} pairs={pairs}", flush=True)
        assert np.array_equal(lib.flat_clusters(dev, N - kept).cpu().numpy(), cut(children.tolist(), N, kept)), kept
    out = torch.empty(N, dtype=torch.int32, device="cuda")
    took, plainly = (least_ms(lambda: lib.flat_clusters(t, 1, out=out)) for t in (dev, plain))
    print(f"  {took * 1000:.0f} us, a plain chain {plainly * 1000:.0f}", flush=True)
    assert took < 20 * plainly, (took, plainly)
