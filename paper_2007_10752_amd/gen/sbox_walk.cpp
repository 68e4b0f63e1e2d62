// Local search that shrinks a 3-input-LUT gate network of a DES S-box (the
// networks and tables are described in sbox_synth.cpp, whose result is the
// usual starting point).
//
// Each move picks a gate v and the input vectors on which v matters (those
// where flipping v changes an output: its observability).  On them v may be
// replaced by
//   - an existing signal or its complement,
//   - one gate over any three signals that do not depend on v, or
//   - two gates: LUT3(w, d, e) for a random pair d, e and a new gate w.
// Unconstrained table entries are filled at random.  Gates that only fed the
// old v (its fanout-free cone) disappear unless the replacement uses them.
// Moves that do not grow the network are taken at once, so the walk drifts
// through networks of equal size; moves that grow it are taken with
// probability exp(-growth / temperature) up to `slack` gates over the best.
// Every accepted network is checked on all 64 inputs.
//
// Built with -DKEYS=n (1..3) the network also takes the key masks of n inputs:
// signals 6 .. 5 + n, each XORed to its input by a gate of the start network.
// That gate counts like the others, so the search saves it where the mask can
// enter a gate that has an operand free (networks.fold_network writes such
// networks out).
//
// Usage: sbox_walk <seconds> <seed> <temperature> <slack> <box table: 64
// values, row-major 4x16> [inputs with key masks] < network.  Prints the
// smallest network found.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>

typedef uint64_t u64;

#ifndef KEYS
#define KEYS 0
#endif
constexpr int kIn = 6 + KEYS;   // inputs: S-box inputs, then key masks
constexpr int kWords = 1 << KEYS;
constexpr int kMax = 56;        // signals of a network: the inputs, then gates
constexpr double kStall = 150;  // seconds without progress before starting over from the best

// A signal's values: bit v of word k for S-box input v under key masks k.
struct Vec {
    u64 w[kWords] = {};
    explicit operator bool() const {
        u64 any = 0;
        for (u64 x : w) any |= x;
        return any != 0;
    }
    bool operator==(const Vec &o) const { return memcmp(w, o.w, sizeof w) == 0; }
    void set(int v, int k) { w[k] |= 1ull << v; }
};
#define VEC_OP(op)                                                  \
    static Vec operator op(const Vec &a, const Vec &b) {            \
        Vec r;                                                      \
        for (int i = 0; i < kWords; i++) r.w[i] = a.w[i] op b.w[i]; \
        return r;                                                   \
    }
VEC_OP(&)
VEC_OP(|)
VEC_OP(^)
static void operator|=(Vec &a, const Vec &b) { a = a | b; }
static Vec operator~(const Vec &a) {
    Vec r;
    for (int i = 0; i < kWords; i++) r.w[i] = ~a.w[i];
    return r;
}

struct Gate {
    int a, b, c, imm;
};
struct Net {
    int n;  // signals
    Gate g[kMax];
    Vec t[kMax];
    int out[4], neg[4];
};

static u64 state;
static u64 rnd() {
    state ^= state << 13;
    state ^= state >> 7;
    state ^= state << 17;
    return state * 0x2545F4914F6CDD1Dull;
}
static int below(int n) { return (int)((rnd() >> 33) % (u64)n); }

static Vec lut(int imm, const Vec &a, const Vec &b, const Vec &c) {
    Vec r;
    for (int i = 0; i < 8; i++)
        if ((imm >> i) & 1) r |= ((i & 4) ? a : ~a) & ((i & 2) ? b : ~b) & ((i & 1) ? c : ~c);
    return r;
}

static Vec target[4];

static bool correct(const Net &n) {
    for (int q = 0; q < 4; q++)
        if (!((n.neg[q] ? ~n.t[n.out[q]] : n.t[n.out[q]]) == target[q])) return false;
    return true;
}

// The live part of gates g[kIn..n), which may be in any order, as a network in
// topological order; false if it is cyclic.
static bool rebuild(const Gate *g, int n, const int *out, const int *neg, Net &r) {
    int map[kMax + 1], seen[kMax + 1] = {};
    struct Frame {
        int v, k;
    } stack[kMax + 8];
    for (int i = 0; i < n; i++) map[i] = i < kIn ? i : -1;
    r.n = kIn;
    for (int q = 0; q < 4; q++) {
        if (map[out[q]] >= 0) continue;
        int sp = 0;
        stack[sp++] = {out[q], 0};
        seen[out[q]] = 1;
        while (sp) {
            Frame &f = stack[sp - 1];
            const Gate &x = g[f.v];
            if (f.k < 3) {
                const int c = f.k == 0 ? x.a : f.k == 1 ? x.b : x.c;
                f.k++;
                if (map[c] < 0) {
                    if (seen[c]) return false;
                    seen[c] = 1;
                    stack[sp++] = {c, 0};
                }
            } else {
                if (r.n >= kMax - 2) return false;
                const Gate y = {map[x.a], map[x.b], map[x.c], x.imm};
                r.g[r.n] = y;
                r.t[r.n] = lut(y.imm, r.t[y.a], r.t[y.b], r.t[y.c]);
                map[f.v] = r.n++;
                sp--;
            }
        }
    }
    for (int q = 0; q < 4; q++) {
        r.out[q] = map[out[q]];
        r.neg[q] = neg[q];
    }
    return true;
}

// Input vectors on which gate v matters; *dep: the signals that depend on v.
static Vec observability(const Net &n, int v, u64 *dep) {
    Vec f[kMax];
    *dep = 1ull << v;
    f[v] = ~n.t[v];
    for (int i = v + 1; i < n.n; i++) {
        const Gate &x = n.g[i];
        if (!(((*dep >> x.a) | (*dep >> x.b) | (*dep >> x.c)) & 1)) continue;
        auto val = [&](int s) { return (*dep >> s) & 1 ? f[s] : n.t[s]; };
        f[i] = lut(x.imm, val(x.a), val(x.b), val(x.c));
        *dep |= 1ull << i;
    }
    Vec care;
    for (int q = 0; q < 4; q++)
        if ((*dep >> n.out[q]) & 1) care |= f[n.out[q]] ^ n.t[n.out[q]];
    return care;
}

// v and the gates that feed nothing but v.
static u64 fanout_free_cone(const Net &n, int v) {
    int refs[kMax] = {};
    auto each = [&](int s, auto f) {
        const Gate &x = n.g[s];
        f(x.a);
        if (x.b != x.a) f(x.b);
        if (x.c != x.a && x.c != x.b) f(x.c);
    };
    for (int i = kIn; i < n.n; i++) each(i, [&](int c) { refs[c]++; });
    for (int q = 0; q < 4; q++) refs[n.out[q]]++;
    u64 cone = 1ull << v;
    int stack[kMax], sp = 0;
    stack[sp++] = v;
    while (sp)
        each(stack[--sp], [&](int c) {
            if (c >= kIn && --refs[c] == 0) {
                cone |= 1ull << c;
                stack[sp++] = c;
            }
        });
    return cone;
}

// Calls f(a, b, c) for every triple of the signals s[0..ns) on which some gate
// is 1 on `on` and 0 on `off`.
template <class F>
static void triples(const Net &n, const int *s, int ns, const Vec &on, const Vec &off, F f) {
    for (int i = 0; i < ns; i++)
        for (int j = i + 1; j < ns; j++) {
            const Vec A = n.t[s[i]], B = n.t[s[j]];
            const Vec cell[4] = {~A & ~B, ~A & B, A & ~B, A & B};
            Vec p[4], z[4];
            int k = 0;
            for (const Vec &m : cell)
                if ((on & m) && (off & m)) {
                    p[k] = on & m;
                    z[k++] = off & m;
                }
            for (int l = j + 1; l < ns; l++) {
                const Vec C = n.t[s[l]];
                bool ok = true;
                for (int q = 0; q < k && ok; q++)
                    ok = !((p[q] & C) && (z[q] & C)) && !((p[q] & ~C) && (z[q] & ~C));
                if (ok) f(s[i], s[j], s[l]);
            }
        }
}

// The table of a gate over (a, b, c) that is 1 on `on` and 0 on `off`, its
// free entries at random.
static int table_of(const Net &n, int a, int b, int c, const Vec &on, const Vec &off) {
    int imm = 0, free = 0;
    for (int i = 0; i < 8; i++) {
        const Vec m = ((i & 4) ? n.t[a] : ~n.t[a]) & ((i & 2) ? n.t[b] : ~n.t[b]) &
                      ((i & 1) ? n.t[c] : ~n.t[c]);
        if (m & on) imm |= 1 << i;
        else if (!(m & off)) free |= 1 << i;
    }
    return imm | (free & below(256));
}

static void print(const Net &n) {
    printf("gates %d\n", n.n - kIn);
    for (int i = kIn; i < n.n; i++)
        printf("g %d %d %d %d %d\n", i, n.g[i].a, n.g[i].b, n.g[i].c, n.g[i].imm);
    for (int q = 0; q < 4; q++) printf("out %d %d %d\n", q, n.out[q], n.neg[q]);
}

int main(int argc, char **argv) {
    if (argc != 5 + 64 + KEYS) {
        fprintf(stderr, "usage: %s seconds seed temperature slack v0 .. v63 [inputs] < network\n", argv[0]);
        return 1;
    }
    const double seconds = atof(argv[1]), temperature = atof(argv[3]);
    state = strtoull(argv[2], 0, 0) * 0x9E3779B97F4A7C15ull + 12345;
    for (int i = 0; i < 20; i++) rnd();
    const int slack = atoi(argv[4]);
    for (int v = 0; v < 64; v++) {
        const int row = ((v >> 5) << 1) | (v & 1), col = (v >> 1) & 15;
        const int val = atoi(argv[5 + row * 16 + col]);
        for (int k = 0; k < kWords; k++) {
            int u = v;  // the raw input that the masks turn into v
            for (int j = 0; j < KEYS; j++)
                if ((k >> j) & 1) u ^= 1 << (5 - atoi(argv[69 + j]));
            for (int q = 0; q < 4; q++)
                if ((val >> (3 - q)) & 1) target[q].set(u, k);
        }
    }
    static Net cur, best, next;
    for (Net *n : {&cur, &next})
        for (int q = 0; q < kIn; q++)
            for (int v = 0; v < 64; v++)
                for (int k = 0; k < kWords; k++)
                    if (q < 6 ? (v >> (5 - q)) & 1 : (k >> (q - 6)) & 1) n->t[q].set(v, k);
    cur.n = kIn;
    auto add = [&](const Gate &x) {
        cur.g[cur.n] = x;
        cur.t[cur.n] = lut(x.imm, cur.t[x.a], cur.t[x.b], cur.t[x.c]);
        return cur.n++;
    };
    int map[kMax];  // signals of the given network, in this one
    for (int q = 0; q < 6; q++) map[q] = q;
    for (int j = 0; j < KEYS; j++) {
        const int q = atoi(argv[69 + j]);
        if (q < 0 || q > 5) return 1;
        map[q] = add({q, 6 + j, 6 + j, 0x3C});
    }
    char line[200];
    while (fgets(line, sizeof line, stdin)) {
        int x, a, b, c, m;
        if (sscanf(line, "g %d %d %d %d %d", &x, &a, &b, &c, &m) == 5 && x >= 6 &&
            x < kMax - 2 - 2 * KEYS && std::min({a, b, c}) >= 0 && std::max({a, b, c}) < x) {
            map[x] = add({map[a], map[b], map[c], m});
        } else if (sscanf(line, "out %d %d %d", &x, &a, &b) == 3 && x >= 0 && x < 4 && a >= 0 && a < kMax - 2) {
            cur.out[x] = map[a];
            cur.neg[x] = b;
        }
    }
    if (!correct(cur)) {
        fprintf(stderr, "the given network is not this S-box\n");
        return 1;
    }
    best = cur;
    const auto t0 = std::chrono::steady_clock::now();
    double progress = 0;
    for (long it = 1;; it++) {
        if (it % 1024 == 0) {
            const double t = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
            if (t > seconds) break;
            if (t - progress > kStall) {
                cur = best;
                progress = t;
            }
        }
        const int v = kIn + below(cur.n - kIn);
        u64 dep;  // (signal set)
        const Vec care = observability(cur, v, &dep);
        const u64 cone = fanout_free_cone(cur, v);
        const int freed = __builtin_popcountll(cone);
        const Vec on = cur.t[v] & care, off = ~cur.t[v] & care;
        int s[kMax], ns = 0;
        for (int i = 0; i < cur.n; i++)
            if (!((dep >> i) & 1)) s[ns++] = i;
        u64 needs[kMax];  // the part of the cone a signal keeps alive
        for (int i = 0; i < cur.n; i++)
            needs[i] = (cone >> i) & 1 ? 1ull << i | needs[cur.g[i].a] | needs[cur.g[i].b] | needs[cur.g[i].c] : 0;
        Gate g[kMax + 1];
        int n = cur.n, out[4], neg[4], delta = 99;
        memcpy(g, cur.g, sizeof cur.g);
        memcpy(out, cur.out, sizeof out);
        memcpy(neg, cur.neg, sizeof neg);
        bool have = false;
        for (int k = 0; k < ns && !have; k++) {
            const int x = s[(k + it) % ns];
            const Vec d = (cur.t[x] ^ cur.t[v]) & care;
            if (d && !(d == care)) continue;
            const int inv = (bool)d;
            for (int i = kIn; i < n; i++) {
                auto swap_in = [&](int &r, int bit) {
                    if (r != v) return;
                    r = x;
                    int imm = 0;
                    for (int e = 0; e < 8; e++)
                        if ((g[i].imm >> (inv ? e ^ bit : e)) & 1) imm |= 1 << e;
                    g[i].imm = imm;
                };
                swap_in(g[i].a, 4);
                swap_in(g[i].b, 2);
                swap_in(g[i].c, 1);
            }
            for (int q = 0; q < 4; q++)
                if (out[q] == v) {
                    out[q] = x;
                    neg[q] ^= inv;
                }
            have = true;
            delta = __builtin_popcountll(needs[x]) - freed;
        }
        // among the replacements, one of those that shrink the network most, or
        // any of those that keep its size
        int pick[3], key = 99;
        long ties = 0;
        auto offer = [&](int a, int b, int c, int d, u64 extra) {
            const int k = std::min(d + __builtin_popcountll((needs[a] | needs[b] | needs[c] | extra) & cone) - freed, 99);
            if (k < key || (k == key && below((int)++ties) == 0)) {
                if (k < key) ties = 1;
                key = k;
                pick[0] = a, pick[1] = b, pick[2] = c;
            }
        };
        if (!have && below(100) < 70) {
            triples(cur, s, ns, on, off, [&](int a, int b, int c) { offer(a, b, c, 1, 0); });
            if (key <= 0) {
                g[v] = {pick[0], pick[1], pick[2], table_of(cur, pick[0], pick[1], pick[2], on, off)};
                have = true;
                delta = key;
            }
        } else if (!have) {
            const int d = s[below(ns)], e = s[below(ns)];
            if (d == e) continue;
            Vec w1, w0;          // where w must be 1, 0
            int outer = 0;       // LUT3(w, d, e)
            for (int cell = 0; cell < 4; cell++) {
                const Vec m = ((cell & 2) ? cur.t[d] : ~cur.t[d]) & ((cell & 1) ? cur.t[e] : ~cur.t[e]);
                if ((on & m) && (off & m)) {
                    const int flip = below(2);
                    w1 |= flip ? off & m : on & m;
                    w0 |= flip ? on & m : off & m;
                    outer |= 1 << (flip ? cell : 4 + cell);
                } else if ((on & m) || (!(off & m) && below(2))) {
                    outer |= 0x11 << cell;
                }
            }
            triples(cur, s, ns, w1, w0, [&](int a, int b, int c) { offer(a, b, c, 2, needs[d] | needs[e]); });
            if (key < 99) {
                g[n] = {pick[0], pick[1], pick[2], table_of(cur, pick[0], pick[1], pick[2], w1, w0)};
                g[v] = {n++, d, e, outer};
                have = true;
                delta = key;
            }
        }
        if (!have) continue;
        if (delta > 0 && (cur.n + delta > best.n + slack ||
                          (double)(rnd() >> 11) / 9007199254740992.0 > exp(-delta / temperature)))
            continue;
        if (!rebuild(g, n, out, neg, next)) continue;
        if (!correct(next)) {
            fprintf(stderr, "verification failed\n");
            return 3;
        }
        cur = next;
        if (cur.n <= best.n) {
            if (cur.n < best.n)
                progress = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
            best = cur;
        }
    }
    print(best);
    return 0;
}
