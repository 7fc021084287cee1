"""The split-BF16 rotation at the widths where its loads change form (multiples of
8, of 4, neither; around a K step of 32) and around its row tiles, against FP64."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim", [1, 7, 8, 12, 24, 31, 32, 40, 63, 64, 72, 100, 104, 300, 768])
def test_split_bf16_rotation(dim):
    """Operands keep 16 bits of significand as hi + lo (2^-17 relative each), lo * lo
    (2^-18) is dropped and FP32 sums K terms: |error| <= (2^-15 + K 2^-23) sum |q p|."""
    import torch
    from paper_2405_12497_amd import rabitq as R
    print(f"[rotation {dim}]", flush=True)
    sys.stdout.flush()
    rng = np.random.default_rng(dim)
    bits = (dim + 63) // 64 * 64
    P = np.linalg.qr(rng.standard_normal((bits, bits)))[0]
    cent = rng.standard_normal((1, dim)).astype(np.float32)
    data = rng.standard_normal((777, dim)).astype(np.float32)
    idx = R.Index(dim, 1, rot_precision=R.RBQ_ROT_BF16X3)
    idx.build_rotation(data, cent, np.zeros(777, np.int32), P)
    P = P[:dim]
    tol = 2.0 ** -15 + dim * 2.0 ** -23

    for nq in (1, 33, 700, 5000):
        q = rng.standard_normal((nq, dim)).astype(np.float32)
        got = R.rbq_debug_rotate(idx.h, torch.from_numpy(q).cuda(), bits).cpu().numpy().astype(np.float64)
        bound = tol * (np.abs(q).astype(np.float64) @ np.abs(P))
        assert (np.abs(got - q.astype(np.float64) @ P) <= bound).all(), nq
    # the residuals of construction: signs, except where the sum is within the bound of 0
    codes = R.rbq_debug_export_codes(idx.h, 777, bits // 64)[0]
    codes = np.asarray(codes).view(np.uint64).reshape(777, bits // 64)
    got = np.unpackbits(codes.view(np.uint8), axis=1, bitorder="little").astype(bool)
    r = (data - cent).astype(np.float64)
    y = r @ P
    bound = tol * (np.abs(r) @ np.abs(P))
    assert ((got == (y > 0)) | (np.abs(y) <= bound)).all()
    idx.close()


@pytest.mark.parametrize("dim,nlist", [(1, 1), (3, 5), (4, 64), (7, 33), (16, 3), (17, 65), (37, 130), (100, 4), (260, 129)])
def test_fp32_rotation_and_centroid_distances(dim, nlist):
    """FP32 products around the tiles (64 rows and columns), K steps of 16 and widths
    that are and are not multiples of 4: sums of K terms, |error| <= (K + 8) 2^-23
    times the sum of the terms' magnitudes."""
    import torch
    from paper_2405_12497_amd import rabitq as R
    print(f"[fp32 {dim} {nlist}]", flush=True)
    rng = np.random.default_rng(dim + nlist)
    bits = (dim + 63) // 64 * 64
    P = np.linalg.qr(rng.standard_normal((bits, bits)))[0]
    cent = rng.standard_normal((nlist, dim)).astype(np.float32)
    data = rng.standard_normal((300, dim)).astype(np.float32)
    idx = R.Index(dim, nlist)
    idx.build_rotation(data, cent, (np.arange(300) % nlist).astype(np.int32), P)
    P, c = P[:dim], cent.astype(np.float64)
    tol = (dim + 8) * 2.0 ** -23
    for nq in (1, 8, 9, 63, 64, 65, 200, 1030):
        q = rng.standard_normal((nq, dim)).astype(np.float32)
        qc, q64 = torch.from_numpy(q).cuda(), q.astype(np.float64)
        got = R.rbq_debug_rotate(idx.h, qc, bits).cpu().numpy()
        assert (np.abs(got - q64 @ P) <= tol * (np.abs(q64) @ np.abs(P))).all(), nq
        d = R.rbq_debug_centroid_dists(idx.h, qc, nlist).cpu().numpy()
        sq, sc = (q64 ** 2).sum(1)[:, None], (c ** 2).sum(1)[None]
        assert (np.abs(d - np.maximum(sq + sc - 2 * q64 @ c.T, 0)) <= tol * (sq + sc + 2 * np.abs(q64) @ np.abs(c.T))).all(), nq
    # searches rotate and score in one launch: every code of every list, exactly
    R.rbq_index_set_eps0(idx.h, 200.0)
    q = rng.standard_normal((70, dim)).astype(np.float32)
    _, got, _ = idx.search(torch.from_numpy(q).cuda(), 5, nlist)
    want = np.sort(((q[:, None].astype(np.float64) - data[None]) ** 2).sum(-1), 1)[:, :5]
    assert (np.abs(got.cpu().numpy() - want) <= want * tol + 1e-12).all()
    idx.close()


@pytest.mark.parametrize("dim,rot", [(64, 0), (100, 0), (100, 1), (768, 0), (768, 1)])
def test_buffers_at_any_float_address(dim, rot):
    """Queries, data and k-means input that begin 4, 8 or 12 bytes past a multiple of
    16, which the kernels read four floats at a time: the results are those of the
    same values at an aligned address."""
    import torch
    from paper_2405_12497_amd import rabitq as R
    print(f"[address {dim} {rot}]", flush=True)
    rng = np.random.default_rng(dim + rot)
    n, nlist, nq = 1300, 24, 700
    data = rng.standard_normal((n, dim)).astype(np.float32)
    q = rng.standard_normal((nq, dim)).astype(np.float32)

    def at(x, shift):
        buf = torch.zeros(x.size + 8, device="cuda")
        v = buf[shift:shift + x.size].view(x.shape)
        v.copy_(torch.from_numpy(x))
        assert v.data_ptr() % 16 == 4 * shift % 16
        return v

    ref = None
    for shift in (0, 1, 2, 3):
        d = at(data, shift)
        cent, assign = R.rbq_kmeans(d, nlist, iters=2, seed=5)
        idx = R.Index(dim, nlist, rot_precision=R.RBQ_ROT_BF16X3 if rot else R.RBQ_ROT_FP32, seed=9)
        idx.build(d, cent, assign)
        out = [cent, assign]
        for m in (1, 5, 40, nq):
            for scan in (R.RBQ_SCAN_POPCNT, R.RBQ_SCAN_MFMA):
                ids, dist, _ = idx.search(at(q[:m], shift), 10, 8, scan_kernel=scan)
                out += [ids, dist]
        torch.cuda.synchronize()
        out = [torch.as_tensor(x).cpu() for x in out]
        ref = ref or out
        for a, b in zip(ref, out):
            assert torch.equal(a, b), shift
        idx.close()
