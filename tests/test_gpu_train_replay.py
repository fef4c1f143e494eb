"""The training of the learned step against a replay in numpy: the same split, initial weights and
minibatch order (std::shuffle and mt19937_64 in a small host program), the same BF16 rounding of
weights, activations and deltas, sums in FP64, the same Adam and cosine rate. The saved weights'
updates agree tensor by tensor, at batches that fill a workgroup of 64 samples, leave one sample
in the last, and end in a minibatch cut short.

Tolerance: Adam turns a gradient into a step of about its sign, so where a gradient nearly cancels
a rounding decides the step, in either program. How much of a tensor that concerns is measured on
the replay itself, as the change of the updates when features and targets move by 2^-18 of their
spread (FP32 logarithms of up to 27 over spreads of 0.6 to 1.2 are good to about 2^-19 of it);
three times the largest of four such changes, and at least 1% of the update's norm, is allowed."""
import math
import os
import shutil
import subprocess

import numpy as np
import pytest

from test_gpu_train_batches import N_PARAMS, samples

K_IN, HID, OUT = 8, 64, 2
SHAPES = [("W1", (K_IN, HID)), ("b1", (HID,)), ("W2", (HID, HID)), ("b2", (HID,)), ("W3", (HID, OUT)), ("b3", (OUT,))]
Y_HE = 0.08

ORDER_CPP = r"""
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <numeric>
#include <random>
#include <vector>
int main(int, char** v)
{
    const size_t m = std::atol(v[1]), n_val = std::atol(v[2]);
    const int seed = std::atoi(v[3]), epochs = std::atoi(v[4]);
    std::vector<uint32_t> order(m);
    std::iota(order.begin(), order.end(), 0u);
    std::mt19937_64 rng((uint32_t)seed);
    std::shuffle(order.begin(), order.end(), rng);
    std::vector<uint32_t> train(order.begin() + n_val, order.end());
    std::fwrite(order.data(), 4, m, stdout);
    const int dims[3][2] = {{8, 64}, {64, 64}, {64, 2}};
    for (auto& d : dims) {
        const float a = std::sqrt(6.0f / (d[0] + d[1]));
        std::uniform_real_distribution<float> u(-a, a);
        for (int i = 0; i < d[0] * d[1]; ++i) {
            const float x = u(rng);
            std::fwrite(&x, 4, 1, stdout);
        }
    }
    for (int e = 0; e < epochs; ++e) {
        std::shuffle(train.begin(), train.end(), rng);
        std::fwrite(train.data(), 4, train.size(), stdout);
    }
}
"""


def bf16(x):
    u = np.ascontiguousarray(x, np.float32).view(np.uint32).astype(np.uint64)
    u = ((u + 0x7FFF + ((u >> 16) & 1)) >> 16) << 16
    return u.astype(np.uint32).view(np.float32).reshape(np.shape(x))


def host_draws(tmp, m, n_val, seed, epochs):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    src, exe = os.path.join(tmp, "order.cpp"), os.path.join(tmp, "order")
    with open(src, "w") as f:
        f.write(ORDER_CPP)
    subprocess.run([cxx, "-O1", "-std=c++17", src, "-o", exe], check=True)
    raw = subprocess.run([exe, str(m), str(n_val), str(seed), str(epochs)], check=True, capture_output=True).stdout
    order, raw = np.frombuffer(raw[:4 * m], np.uint32), raw[4 * m:]
    w = {}
    for k, shape in SHAPES:
        if k[0] == "W":
            n = shape[0] * shape[1]
            w[k], raw = np.frombuffer(raw[:4 * n], np.float32).reshape(shape), raw[4 * n:]
        else:
            w[k] = np.zeros(shape, np.float32)
    return order, w, np.frombuffer(raw, np.uint32).reshape(epochs, m - n_val)


def features_and_targets(X, Y, y_he):
    """The inputs' logarithms, and the targets' distance from the exponential relaxation of x_HI
    (Hui & Gnedin 1997 case-B recombination and collisional ionisation of hydrogen)."""
    x = X.astype(np.float64)
    F = np.stack([np.log10(x[:, 0]), x[:, 1], np.log10(x[:, 2]), np.log10(np.maximum(x[:, 3], 1e-30)),
                  np.log10(x[:, 4]), np.log10(np.maximum(x[:, 5], 1e-35)), x[:, 6], x[:, 7]], 1)
    T = x[:, 2]
    lam = 2.0 * 157807.0 / T
    alpha = 2.753e-14 * lam ** 1.5 / (1.0 + (lam / 2.740) ** 0.407) ** 2.242
    k_hi = 21.11 * T ** -1.5 * np.exp(-lam / 2) * lam ** -1.089 / (1.0 + (lam / 0.354) ** 0.874) ** 1.101
    ne = x[:, 0] * ((1.0 - x[:, 1]) + y_he * (x[:, 6] + 2.0 * np.maximum(0.0, 1.0 - x[:, 7] - x[:, 6])))
    a, b = alpha * ne, x[:, 3] + k_hi * ne
    xeq = a / (a + b)
    base = xeq + (x[:, 1] - xeq) * np.exp(-(a + b) * x[:, 4])
    return F, np.stack([Y[:, 0] - base, np.log10(Y[:, 1].astype(np.float64)) - np.log10(T)], 1)


def standardised(v, train):
    mu, sd = v[train].mean(0), np.sqrt(np.maximum(1e-12, v[train].var(0)))
    return (v - mu) / sd


def gradient(w, F, T):
    """Sums over a minibatch of the loss's gradients, through BF16 weights, activations and deltas."""
    W1, W2, W3 = (bf16(w[k]).astype(np.float64) for k in ("W1", "W2", "W3"))
    x = bf16(F).astype(np.float64)
    h1 = bf16(np.maximum((x @ W1 + w["b1"]).astype(np.float32), 0)).astype(np.float64)
    h2 = bf16(np.maximum((h1 @ W2 + w["b2"]).astype(np.float32), 0)).astype(np.float64)
    o = h2 @ W3 + w["b3"]
    do = bf16((2.0 * (o - T)).astype(np.float32)).astype(np.float64)
    d2 = bf16(np.where(h2 > 0, do @ W3.T, 0).astype(np.float32)).astype(np.float64)
    d1 = bf16(np.where(h1 > 0, d2 @ W2.T, 0).astype(np.float32)).astype(np.float64)
    return {"W1": x.T @ d1, "b1": d1.sum(0), "W2": h1.T @ d2, "b2": d2.sum(0), "W3": h2.T @ do, "b3": do.sum(0)}


def replay(F, T, w0, orders, batch, lr, gradient=gradient):
    w = {k: v.astype(np.float32) for k, v in w0.items()}
    m1 = {k: np.zeros_like(v) for k, v in w.items()}
    m2 = {k: np.zeros_like(v) for k, v in w.items()}
    n, step, f = orders.shape[1], 0, np.float32
    total = orders.shape[0] * ((n + batch - 1) // batch)
    for order in orders:
        for first in range(0, n, batch):
            idx = order[first:first + batch]
            rate = f(lr * (0.05 + 0.95 * 0.5 * (1.0 + math.cos(math.pi * step / total))))
            step += 1
            g = gradient(w, F[idx], T[idx])
            for k in w:
                gk = (g[k] / len(idx)).astype(np.float32)
                m1[k] = f(0.9) * m1[k] + f(0.1) * gk
                m2[k] = f(0.999) * m2[k] + f(0.001) * gk * gk
                mh, vh = m1[k] / f(1 - 0.9 ** step), m2[k] / f(1 - 0.999 ** step)
                w[k] = w[k] - rate * mh / (np.sqrt(vh) + f(1e-8))
    return w


def setup(tmp, m, batch, epochs, seed):
    X, Y = samples(m, m + batch)
    n_val = max(64, int(0.1 * m))
    order, w0, orders = host_draws(tmp, m, n_val, seed, epochs)
    F, T = features_and_targets(X, Y, Y_HE)
    train = order[n_val:]
    return X, Y, standardised(F, train).astype(np.float32), standardised(T, train), w0, orders


def distance(a, b, w0):
    """Per tensor, the distance of two trained networks in units of the update's norm."""
    return {k: float(np.linalg.norm(a[k] - b[k]) / np.linalg.norm(b[k] - w0[k])) for k, _ in SHAPES}


def tolerance(F, T, w0, orders, batch, lr, ref):
    worst = {k: 0.0 for k, _ in SHAPES}
    for s in range(4):
        rng = np.random.default_rng(s)
        moved = replay((F + rng.uniform(-1, 1, F.shape) * 2.0 ** -18).astype(np.float32),
                       T + rng.uniform(-1, 1, T.shape) * 2.0 ** -18, w0, orders, batch, lr)
        for k, d in distance(moved, ref, w0).items():
            worst[k] = max(worst[k], d)
    return {k: max(0.01, 3.0 * v) for k, v in worst.items()}


CASES = [(1024, 64, 1), (1024, 65, 1), (1100, 129, 2), (2000, 1900, 6)]


@pytest.mark.gpu
@pytest.mark.parametrize("m,batch,epochs", CASES)
def test_weights_follow_the_replay(arc, tmp_path, m, batch, epochs):
    import torch

    X, Y, F, T, w0, orders = setup(str(tmp_path), m, batch, epochs, 7)
    ref = replay(F, T, w0, orders, batch, 2e-3)
    tol = tolerance(F, T, w0, orders, batch, 2e-3, ref)
    ctx = arc.Context(0)
    try:
        net = arc.MLP(ctx)
        net.train(torch.from_numpy(X).cuda(), torch.from_numpy(Y).cuda(), epochs=epochs, batch=batch, lr=2e-3, seed=7,
                  val_frac=0.1, y_he=Y_HE, collisional=1)
        flat = np.frombuffer(net.save()[-4 * N_PARAMS:], np.float32)
        net.close()
    finally:
        ctx.close()
    got, at = {}, 0
    for k, shape in SHAPES:
        n = int(np.prod(shape))
        got[k], at = flat[at:at + n].reshape(shape), at + n
    d = distance(got, ref, w0)
    print({k: (round(d[k], 5), round(tol[k], 5)) for k in d})
    assert all(d[k] <= tol[k] for k in d), (d, tol)


def planted(kind):
    """A replay's gradient with a mistake in it."""
    def wrong(w, F, T):
        if kind == "last sample lost":
            g = gradient(w, F[:-1], T[:-1])
        elif kind == "last sample twice":
            g = gradient(w, np.concatenate([F, F[-1:]]), np.concatenate([T, T[-1:]]))
        else:
            g = gradient(w, F, T)
        if kind == "dW1 tiles swapped":
            g["W1"] = np.concatenate([g["W1"][:, 16:32], g["W1"][:, :16], g["W1"][:, 32:]], 1)
        if kind == "dW3 columns swapped":
            g["W3"] = g["W3"][:, ::-1]
        if kind == "b1 sums of half":
            W = gradient(w, F[:len(F) // 2], T[:len(T) // 2])
            g["b1"] = W["b1"]
        return g
    return wrong


@pytest.mark.parametrize("kind,tensors", [
    ("last sample lost", ["W1", "W2", "W3"]), ("last sample twice", ["W1", "W2", "W3"]), ("dW1 tiles swapped", ["W1"]),
    ("dW3 columns swapped", ["W3"]), ("b1 sums of half", ["b1"])])
def test_the_tolerance_tells_mistakes(tmp_path, kind, tensors):
    m, batch, epochs = CASES[1]
    _, _, F, T, w0, orders = setup(str(tmp_path), m, batch, epochs, 7)
    ref = replay(F, T, w0, orders, batch, 2e-3)
    tol = tolerance(F, T, w0, orders, batch, 2e-3, ref)
    d = distance(replay(F, T, w0, orders, batch, 2e-3, planted(kind)), ref, w0)
    print(kind, {k: (round(d[k], 4), round(tol[k], 4)) for k in d})
    assert all(d[k] > 2.0 * tol[k] for k in tensors), (d, tol)
