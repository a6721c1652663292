"""A class's rounds end with its last step, whatever the chunk length: the bits,
step counts and times of a solve alone, over chunks of even and odd length that
end before, at and long after the solves, polled at once or only at the end."""
import numpy as np
import pytest

from test_gpu_omega1 import state1d, state2d

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("late_poll", [False, True])
@pytest.mark.parametrize("chunk", [1, 2, 3, 7, 16, 33, 64])
def test_chunks_of_any_length_give_the_bits_of_a_solve_alone(gpu, chunk, late_poll):
    reqs = [state1d("euler", 700, 1, max_steps=0), state1d("euler", 300, 2, max_steps=1), state1d("sw", 900, 3, max_steps=40),
            state1d("euler", 500, 4, max_steps=33, omega=1.4), state2d("euler", 70, 30, 5, max_steps=17),
            state2d("mhd", 40, 20, 6, max_steps=32, omega=1.3), state2d("sw", 50, 20, 7, T=0.01)]
    ref = []
    for P in reqs:
        s = gpu.Solver(P, precision="fp32")
        s.init()
        ref.append(s.run())
        s.close()
    assert ref[-1][2] > 3
    pool = gpu.Pool(1 << 27, "fp32")
    got = {}
    for rep in range(2):  # the second batch starts at another round
        for i, P in enumerate(reqs):
            pool.submit(P, tag=rep * 100 + i)
        for _ in range(200 // chunk if late_poll else 1000):
            pool.run(chunk)
            if not late_poll:
                for c in pool.poll():
                    got[c["tag"]] = c
                if len(got) == (rep + 1) * len(reqs):
                    break
        for c in pool.poll():
            got[c["tag"]] = c
    pool.close()
    assert len(got) == 2 * len(reqs)
    for tag, c in got.items():
        U, t, n = ref[tag % 100]
        assert c["status"] == 0 and c["steps"] == n and c["t"] == t and np.array_equal(c["U"], U), tag
