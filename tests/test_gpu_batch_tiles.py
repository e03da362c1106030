"""Tiles of batched plans: the tile size that plans of large extracts take, with
small tiles, so that small covers reach it; results against the oracle byte for
byte."""
import numpy as np
import pytest
import torch

import oracle
from paper_0912_0947_amd import batch, inputs
from paper_0912_0947_amd._lib import JOB_RAW, OK, OP_EXTRACT

from gpu_helpers import DEV, assert_bytes_equal, to_host

pytestmark = pytest.mark.gpu


@pytest.fixture
def restore_tiles():
    saved = batch.tune_state()
    yield
    batch.tune_restore(saved)


@pytest.mark.parametrize("block", [128, 1024])
@pytest.mark.parametrize("raw", [False, True])
@pytest.mark.parametrize("count,total", [(60, 524288), (60, 524287), (256, 524288), (257, 526335)])
def test_tiles_of_large_extracts(count, total, raw, block, restore_tiles):
    """Plans of extracts take tiles of 8 embed tiles from 4 such tiles a job
    on average and 1024 of them in all (tiles of 64 vectors here: 2048 vectors
    a job, 524,288 in all), else of 2: on the lines, one vector below either,
    jobs around the tile sizes, blocks of twice the threads and of the most a
    block may have."""
    batch.tune_set(block, 1, 0, 0, 64)
    g = inputs.rng(4491, count, total)
    v = np.concatenate([[4, 63, 128, 129, 511, 512, 513, 1024, 1025], g.integers(1, 2 * total // count, size=count - 10)])
    v = np.floor(v * min(1.0, (total - 3000) / v.sum())).astype(np.int64).clip(2)
    v = np.append(v, total - v.sum())
    assert v.size == count and v.sum() == total and v.min() > 1
    tile = 512 if total >= 2048 * count and total >= 524288 else 128
    jobs = batch.make_jobs(count)
    jobs["k"] = k = 1 + np.arange(count) % 8
    size = 2 * k * v - g.integers(0, 2 * k)  # stream bytes that end in the job's last vector
    size = np.maximum(size, 4)
    jobs["n"] = 16 * v + g.integers(0, 40, size=count)
    offs = np.concatenate([[0], np.cumsum([batch.align_up(int(x)) for x in jobs["n"]])])
    mo = np.concatenate([[0], np.cumsum([batch.align_up(int(x)) for x in size])])
    jobs["stego_off"], jobs["msg_off"], jobs["op"] = offs[:-1], mo[:-1], OP_EXTRACT
    want = np.full(int(mo[-1]), 0x33, np.uint8)
    stego = np.zeros(int(offs[-1]), np.uint8)
    for i in range(count):
        o, n, kk, ln = int(offs[i]), int(jobs["n"][i]), int(k[i]), int(size[i]) - (0 if raw else 4)
        msg = inputs.random_bytes(ln, 4492, i)
        cover = inputs.random_bytes(n, 4493, i)
        rc, stego[o:o + n] = oracle.embed_raw(cover, 0, msg, 8 * ln, kk) if raw else oracle.embed(cover, msg, kk)
        assert rc == OK
        want[mo[i]:mo[i] + ln] = msg
    if raw:
        jobs["flags"], jobs["stream_bits"] = JOB_RAW, 8 * size
    else:
        jobs["msg_cap"] = size - 4
    out = torch.full((want.size,), 0x33, dtype=torch.uint8, device=DEV)
    status = torch.full((count,), 99, dtype=torch.int32, device=DEV)
    lens = torch.full((count,), -1, dtype=torch.int32, device=DEV)
    plan = batch.Plan(count, OP_EXTRACT, jobs)
    try:
        assert plan.tiles == int((-(-v // tile)).sum())
        plan.extract_batch(torch.from_numpy(stego).to(DEV), out, lens, status)
        assert_bytes_equal(to_host(out), want, "extracts of %d vectors" % total)
    finally:
        plan.close()
    assert (status.cpu().numpy() == OK).all()
    assert (lens.cpu().numpy() == (0 if raw else size - 4)).all()
