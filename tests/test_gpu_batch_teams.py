"""Start teams of the batched solve: a problem that would outlast the others starts with several
workgroups. Sizes sit at the edges of the member limit (16 tiles of 64 rows a member;
16 members at most) and on both sides of 16 columns; the results match those of one workgroup. And the
row lengths that the matrix product meets."""
import threading

import numpy as np
import pytest

from paper_2306_10379_amd import inputs as I

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def _solver(sides, ps, precision="fp64"):
    from paper_2306_10379_amd import gsi
    mats = [I.schrodinger_2d(N, I.random_wells(900 + N, count=(4, 6))) for N in sides]
    X0s = [I.start_block(A.n, p, 901) for A, p in zip(mats, ps)]
    return gsi.BatchedSolver(mats, X0s, ps, which=-1, precision=precision, tol=1e-10, max_iter=20000)


def _solve(b):
    _, iters, status = b.solve()
    *_, team = b.timeline()
    assert np.all(status == 1)
    return [b.results(i)[0] for i in range(len(b.ps))], team


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("sides,ps", [
    ([45], [5]),                 # 2025 rows, 32 tiles: two members
    ([44], [5]),                 # 1936 rows, 31 tiles: one
    ([130], [17]),               # 265 tiles: the most members
    ([96, 12, 11], [20, 3, 4]),  # one problem that decides the end among small ones
], ids=["two", "one", "most", "among"])
def test_start_teams_match_one_workgroup(sides, ps, precision):
    """Both solves end below rho = 1e-10, where Ritz values are exact to rho^2 ||A||^2 / gap, far
    below the 1e-10 asked for here."""
    with _solver(sides, ps, precision) as b:
        print(f"teams {sides} {ps} {precision}", flush=True)
        got, team = _solve(b)
        tiles = [(N * N + 63) // 64 for N in sides]
        assert all(t <= max(1, min(16, n // 16)) for t, n in zip(team, tiles)), team
        assert team[0] == max(1, min(16, tiles[0] // 16)) and np.all(team[1:] == 1), team
        b.set_tuning(1 << 20, 1, 1 << 20)
        ref, team = _solve(b)
        assert np.all(team == 1)
        for x, y in zip(got, ref):
            assert np.max(np.abs(x - y) / np.abs(y)) <= 1e-10


def test_start_teams_follow_the_tiles_per_member():
    """A changed limit sizes the start teams anew, up and down (32 tiles: one member per limit)."""
    with _solver([45], [5]) as b:
        ref, team = _solve(b)
        assert team[0] == 2
        for limit, want in ((4, 8), (8, 4), (32, 1), (16, 2)):
            b.set_tuning(limit, 1, 1 << 20)  # no recruiting
            got, team = _solve(b)
            assert team[0] == want, (limit, team)
            assert np.max(np.abs(got[0] - ref[0]) / np.abs(ref[0])) <= 1e-10


def test_every_solve_follows_the_limit_set_before_it():
    """Limits set and solves launched one after the other on a stream that the default stream does
    not wait for: queue, teams and control block belong together in every one of them."""
    from paper_2306_10379_amd import gsi
    sides, ps = [45, 64, 20, 33], [5, 9, 4, 20]
    tiles = [(N * N + 63) // 64 for N in sides]
    mats = [I.schrodinger_2d(N, I.random_wells(900 + N, count=(4, 6))) for N in sides]
    X0s = [I.start_block(A.n, p, 901) for A, p in zip(mats, ps)]
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        b = gsi.BatchedSolver(mats, X0s, ps, which=-1, precision="fp64", max_iter=3)
        for k in range(40):
            limit = (4, 8, 16, 32, 1 << 20)[k % 5]
            b.set_tuning(limit, 1, 1 << 20)
            _, iters, status = b.solve()
            *_, team = b.timeline()
            assert np.all(iters == 3) and np.all(status == 2)
            assert all(t <= max(1, min(16, n // limit)) for t, n in zip(team, tiles)), (limit, team)
            if limit == 1 << 20:
                assert np.all(team == 1)
        torch.cuda.synchronize()


def test_start_teams_of_two_solvers_at_once():
    """Two launches share the device; each closes its teams with whoever arrives."""
    with _solver([96, 90, 20], [12, 20, 4]) as a, _solver([80, 100], [18, 9]) as b:
        ref = [_solve(s)[0] for s in (a, b)]
        out = [None, None]

        def run(k, s):
            out[k] = _solve(s)[0]

        for _ in range(3):
            ts = [threading.Thread(target=run, args=(k, s)) for k, s in enumerate((a, b))]
            [t.start() for t in ts]
            [t.join() for t in ts]
            for k in range(2):
                for x, y in zip(out[k], ref[k]):
                    assert np.max(np.abs(x - y) / np.abs(y)) <= 1e-10


@pytest.mark.parametrize("p", [5, 20])
@pytest.mark.parametrize("n", [64, 77, 1100])
def test_row_lengths_of_the_matrix_product(n, p):
    """Rows of seven nonzeros (the most that a batch takes: 112 in a wave's 16 rows), of one, of
    none and of lengths that differ within the 16, against dense eigenvalues."""
    from paper_2306_10379_amd import gsi
    a = np.zeros((n, n))
    for i in range(33):  # band of seven, then short rows
        for j in range(max(0, i - 3), min(33, i + 4)):
            a[i, j] = 40.0 + 2.0 * i if i == j else 1.0 / (1 + abs(i - j))
    a[np.arange(40, n), np.arange(40, n)] = np.linspace(1.0, 3.0, n - 40)  # rows 33 .. 39 are empty
    for i in range(45, n - 1, 2):
        a[i, i + 1] = a[i + 1, i] = 0.5
    A = I.dense_to_csr(a)
    lens = np.diff(A.rowptr)
    assert lens.max() == 7 and lens.min() == 0
    print(f"rows {n} {p} nnz {A.nnz}", flush=True)
    with gsi.BatchedSolver([A], [I.start_block(n, p, 5)], [p], which=1, precision="fp64", tol=1e-11,
                           max_iter=20000) as b:
        ritz, _ = _solve(b)
    w = np.linalg.eigvalsh(a)[::-1][:p]
    assert np.max(np.abs(ritz[0] - w)) <= 1e-10 * np.max(np.abs(w))


def test_longer_rows_are_refused_by_name():
    """A valid matrix with one row of eight nonzeros among shorter ones: refused, as it has no room
    in the product's buffer, and the message says so. The same matrix solves on its own."""
    from paper_2306_10379_amd import gsi
    n, p = 200, 4
    a = np.diag(np.linspace(1.0, 5.0, n))
    a[100, 20:27] = a[20:27, 100] = 0.1
    A = I.dense_to_csr(a)
    assert np.diff(A.rowptr).max() == 8
    X0 = I.start_block(n, p, 5)
    with pytest.raises(gsi.GsiError, match="problem 1: a row of more than 7 nonzeros") as e:
        gsi.BatchedSolver([I.dense_to_csr(np.diag(np.linspace(1.0, 5.0, n))), A], [X0, X0], [p, p], which=1)
    assert e.value.status == gsi.GSI_EINVAL
    with gsi.Solver(A, X0, p, tol=1e-10) as s:
        ritz = s.run().ritz
    w = np.linalg.eigvalsh(a)[::-1][:p]
    assert np.max(np.abs(ritz - w)) <= 1e-10 * np.max(np.abs(w))
